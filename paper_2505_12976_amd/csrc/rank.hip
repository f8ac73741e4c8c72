// Winners and ranking from the closure p (Section 2.1): y beats x iff
// p[y][x] > p[x][y]; x is a Schulze winner iff nobody beats it; the ranking
// orders candidates by how many candidates beat them, then by id.
#include "internal.h"
#include "tile_io.h"

namespace {

// beaten_by[x] += #{y : p[y][x] > p[x][y]} over one pair of 64 x 64 blocks
// of candidates (X, Y), X <= Y: both directions need the same two tiles of
// p, so p is read once.
template <typename E>
__global__ __launch_bounds__(256) void k_beaten_by(const E *__restrict__ p, int64_t ldp, int32_t m,
                                                   int32_t *__restrict__ beaten) {
    __shared__ E py[64][65];  // py[a][b] = p[Y0 + a][X0 + b]
    __shared__ E px[64][65];  // px[a][b] = p[X0 + a][Y0 + b]
    if (blockIdx.x > blockIdx.y) return;
    const int32_t X0 = blockIdx.x * 64, Y0 = blockIdx.y * 64;
    tio::load<E>(py, p, ldp, Y0, X0, m, m);
    tio::load<E>(px, p, ldp, X0, Y0, m, m);
    __syncthreads();
    const int l = threadIdx.x & 63, part = threadIdx.x >> 6;
    int32_t cx = 0, cy = 0;
    for (int o = part * 16; o < part * 16 + 16; ++o) {
        cx += py[o][l] > px[l][o] ? 1 : 0;  // y = Y0 + o beats x = X0 + l
        cy += px[o][l] > py[l][o] ? 1 : 0;  // x = X0 + o beats y = Y0 + l
    }
    if (cx && X0 + l < m) atomicAdd(&beaten[X0 + l], cx);
    if (X0 != Y0 && cy && Y0 + l < m) atomicAdd(&beaten[Y0 + l], cy);
}

// One workgroup: the winners and their number (nothing to clear first).
__global__ __launch_bounds__(1024) void k_winners(const int32_t *__restrict__ beaten, int32_t m,
                                                  uint8_t *__restrict__ is_winner, int32_t *__restrict__ n_winners) {
    __shared__ int32_t part[16];
    int32_t n = 0;
    for (int32_t x = threadIdx.x; x < m; x += 1024) {
        const bool w = beaten[x] == 0;
        is_winner[x] = w ? 1 : 0;
        n += w ? 1 : 0;
    }
    for (int off = 32; off >= 1; off >>= 1) n += __shfl_xor(n, off);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0 && n_winners) {
        for (int g = 1; g < 16; ++g) n += part[g];
        n_winners[0] = n;
    }
}

// Small elections (m <= RANK_SMALL): p in one workgroup's LDS, the beaten-by
// counts, and whatever of winners and ranking is asked for, in one launch
// (the separate kernels take three launches of about 4.5 us each, most of it
// the launch).  Eight threads per candidate.
constexpr int RANK_SMALL = 128;
template <typename E>
__global__ __launch_bounds__(1024) void k_rank_small(const E *__restrict__ p, int64_t ldp, int32_t m,
                                                     uint8_t *__restrict__ is_winner, int32_t *__restrict__ n_winners,
                                                     int32_t *__restrict__ order, int32_t *__restrict__ beaten_by) {
    __shared__ E q[RANK_SMALL][RANK_SMALL + 1];
    __shared__ int32_t key[RANK_SMALL];
    __shared__ int32_t wins;
    if (threadIdx.x == 0) wins = 0;
    for (int r = threadIdx.x >> 7; r < m; r += 8) {
        const int c = threadIdx.x & 127;
        if (c < m) q[r][c] = p[(int64_t)r * ldp + c];
    }
    __syncthreads();
    const int x = threadIdx.x >> 3, part = threadIdx.x & 7;
    int32_t b = 0;
    if (x < m)
        for (int y = part; y < m; y += 8) b += q[y][x] > q[x][y] ? 1 : 0;
    for (int off = 4; off >= 1; off >>= 1) b += __shfl_xor(b, off);
    if (x < m && part == 0) {
        key[x] = b * m + x;
        if (beaten_by) beaten_by[x] = b;
        if (is_winner) {
            is_winner[x] = b == 0 ? 1 : 0;
            if (b == 0) atomicAdd(&wins, 1);
        }
    }
    __syncthreads();
    if (order) {
        int32_t r = 0;
        if (x < m)
            for (int y = part; y < m; y += 8) r += key[y] < key[x] ? 1 : 0;
        for (int off = 4; off >= 1; off >>= 1) r += __shfl_xor(r, off);
        if (x < m && part == 0) order[r] = x;
    }
    if (n_winners && threadIdx.x == 0) n_winners[0] = wins;
}

int rank_small(schulze_ctx *ctx, hipStream_t s, int kid, const void *p, int64_t ldp, int32_t m, int dtype,
               uint8_t *is_winner, int32_t *n_winners, int32_t *order, int32_t *beaten_by) {
    if (dtype == SCHULZE_U16)
        SCHULZE_LAUNCH(ctx, kid, s,
                       k_rank_small<uint16_t><<<dim3(1), dim3(1024), 0, s>>>(static_cast<const uint16_t *>(p), ldp, m,
                                                                             is_winner, n_winners, order, beaten_by));
    else
        SCHULZE_LAUNCH(ctx, kid, s,
                       k_rank_small<int32_t><<<dim3(1), dim3(1024), 0, s>>>(static_cast<const int32_t *>(p), ldp, m,
                                                                            is_winner, n_winners, order, beaten_by));
    return SCHULZE_OK;
}

// order[rank(x)] = x with rank(x) = #{y : (beaten[y], y) < (beaten[x], x)}.
// Keys beaten*m + id are distinct and fit 32 bits for m <= 65535.  A
// workgroup takes RS_X candidates; its RS_G wavefronts count over
// interleaved shares of the keys (staged in LDS RS_CHUNK at a time, each
// read a broadcast) and the shares are summed in LDS.  (One thread per
// candidate over every key left most of the chip idle.)
constexpr int RS_X = 64;
constexpr int RS_G = 16;
constexpr int RS_CHUNK = 4096;
__global__ __launch_bounds__(64 * RS_G) void k_rank_sort(const int32_t *__restrict__ beaten, int32_t m,
                                                         int32_t *__restrict__ order) {
    __shared__ uint32_t keys[RS_CHUNK];
    __shared__ int32_t part[RS_G][RS_X];
    const int xl = threadIdx.x & 63, grp = threadIdx.x >> 6;
    const int32_t x = blockIdx.x * RS_X + xl;
    auto key = [&](int32_t y) { return (uint32_t)beaten[y] * (uint32_t)m + (uint32_t)y; };
    const uint32_t kx = x < m ? key(x) : 0xFFFFFFFFu;
    int32_t rank = 0;
    for (int32_t y0 = 0; y0 < m; y0 += RS_CHUNK) {
        __syncthreads();
        for (int i = threadIdx.x; i < RS_CHUNK; i += 64 * RS_G) keys[i] = y0 + i < m ? key(y0 + i) : 0xFFFFFFFFu;
        __syncthreads();
        const int lim = min(RS_CHUNK, m - y0);
        for (int i = grp; i < lim; i += RS_G) rank += keys[i] < kx ? 1 : 0;
    }
    part[grp][xl] = rank;
    __syncthreads();
    if (grp == 0 && x < m) {
        int32_t r = 0;
        for (int g = 0; g < RS_G; ++g) r += part[g][xl];
        order[r] = x;
    }
}

template <typename E>
int beaten_by(schulze_ctx *ctx, hipStream_t s, const E *p, int64_t ldp, int32_t m, int32_t *beaten) {
    int rc = fill_u32(ctx, s, reinterpret_cast<uint32_t *>(beaten), (size_t)m, 0u);
    if (rc != SCHULZE_OK) return rc;
    dim3 grid((unsigned)ceil_div(m, 64), (unsigned)ceil_div(m, 64));
    SCHULZE_LAUNCH(ctx, K_BEATEN_BY, s, k_beaten_by<E><<<grid, dim3(256), 0, s>>>(p, ldp, m, beaten));
    return SCHULZE_OK;
}

int beaten_any(schulze_ctx *ctx, hipStream_t s, const void *p, int64_t ldp, int32_t m, int dtype,
               int32_t *beaten) {
    if (dtype == SCHULZE_U16) return beaten_by(ctx, s, static_cast<const uint16_t *>(p), ldp, m, beaten);
    return beaten_by(ctx, s, static_cast<const int32_t *>(p), ldp, m, beaten);
}

int check_args(schulze_ctx *ctx, const void *p, int64_t ldp, int32_t m, int dtype) {
    if (!ctx || !p) return SCHULZE_EINVAL;
    if (m < 1 || ldp < m) return SCHULZE_EINVAL;
    if (dtype != SCHULZE_U16 && dtype != SCHULZE_I32) return SCHULZE_EINVAL;
    if (m > 65535) return SCHULZE_EUNSUPPORTED;
    return bind_device(ctx);
}

}  // namespace

extern "C" int schulze_winners(schulze_ctx *ctx, void *stream, const void *p, int64_t ldp, int32_t m, int dtype,
                               uint8_t *is_winner, int32_t *n_winners) {
    int rc = check_args(ctx, p, ldp, m, dtype);
    if (rc != SCHULZE_OK) return rc;
    if (!is_winner) return SCHULZE_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    if (m <= RANK_SMALL) return rank_small(ctx, s, K_WINNERS, p, ldp, m, dtype, is_winner, n_winners, nullptr, nullptr);
    if ((rc = ws_reserve(ctx, WS_RANK, sizeof(int32_t) * (size_t)m)) != SCHULZE_OK) return rc;
    int32_t *beaten = static_cast<int32_t *>(ctx->ws[WS_RANK]);
    if ((rc = beaten_any(ctx, s, p, ldp, m, dtype, beaten)) != SCHULZE_OK) return rc;
    SCHULZE_LAUNCH(ctx, K_WINNERS, s, k_winners<<<dim3(1), dim3(1024), 0, s>>>(beaten, m, is_winner, n_winners));
    return SCHULZE_OK;
}

extern "C" int schulze_ranking(schulze_ctx *ctx, void *stream, const void *p, int64_t ldp, int32_t m, int dtype,
                               int32_t *order, int32_t *beaten_by_out) {
    int rc = check_args(ctx, p, ldp, m, dtype);
    if (rc != SCHULZE_OK) return rc;
    if (!order) return SCHULZE_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    if (m <= RANK_SMALL) return rank_small(ctx, s, K_RANK_SORT, p, ldp, m, dtype, nullptr, nullptr, order, beaten_by_out);
    int32_t *beaten = beaten_by_out;
    if (!beaten) {
        if ((rc = ws_reserve(ctx, WS_RANK, sizeof(int32_t) * (size_t)m)) != SCHULZE_OK) return rc;
        beaten = static_cast<int32_t *>(ctx->ws[WS_RANK]);
    }
    if ((rc = beaten_any(ctx, s, p, ldp, m, dtype, beaten)) != SCHULZE_OK) return rc;
    SCHULZE_LAUNCH(ctx, K_RANK_SORT, s,
                   k_rank_sort<<<dim3((unsigned)ceil_div(m, RS_X)), dim3(64 * RS_G), 0, s>>>(beaten, m, order));
    return SCHULZE_OK;
}
