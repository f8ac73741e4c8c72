// Learned winner proposer: a 16 -> 128 -> 128 -> 1 ReLU network over the
// per-candidate features, with hand-written BF16 MFMA GEMMs (FP32
// accumulation) for the forward pass, the backward pass and a segmented
// softmax loss over elections, plus Adam with FP32 master weights.
//
// Parameter layout (FP32, SCHULZE_MLP_PARAMS floats):
//   W1[16][128] | b1[128] | W2[128][128] | b2[128] | W3[128] | b3[1]
// z1 = x W1 + b1, h1 = relu(z1), z2 = h1 W2 + b2, h2 = relu(z2), s = h2 W3 + b3.
// Rounding points (the CPU reference applies the same ones): x, W1, W2, W3,
// h1, h2, dz2 and dz1 are rounded to BF16 (nearest even); products are
// accumulated in FP32; biases stay FP32.
//
// MFMA lane layouts on gfx950 (checked on the device):
//   v_mfma_f32_32x32x16_bf16: lane l supplies A row l%32 / B column l%32 with
//   k = 8 (l/32) + e, e < 8; D element i of lane l is row 8 (i/4) + 4 (l/32)
//   + i%4, column l%32.
//   v_mfma_f32_16x16x32_bf16: lane l supplies row/column l%16 with
//   k = 8 (l/16) + e; D element i of lane l is row 4 (l/16) + i, column l%16.
#include "internal.h"

namespace {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NF = 16, NH = 128;
constexpr int OFF_W1 = 0, OFF_B1 = OFF_W1 + NF * NH, OFF_W2 = OFF_B1 + NH, OFF_B2 = OFF_W2 + NH * NH,
              OFF_W3 = OFF_B2 + NH, OFF_B3 = OFF_W3 + NH, NPARAM = OFF_B3 + 1;
constexpr int ROWS = 64;            // rows per tile
constexpr int PH = NH + 8;          // padded LDS pitch (bf16) of 128-wide rows
constexpr int PF = NF + 8;          // padded pitch of 16-wide rows
constexpr int PR = ROWS + 8;        // padded pitch of 64-wide (row index) rows

__device__ inline bf16 to_bf16(float f) { return (bf16)f; }
__device__ inline float from_bf16(bf16 b) { return (float)b; }

__device__ inline bf16x8 ld8(const bf16 *p) { return *reinterpret_cast<const bf16x8 *>(p); }

// BF16 copies of the weights in the layouts the kernels read:
// w1t[j][f] = W1[f][j], w2t[j][i] = W2[i][j], w2[i][j] = W2[i][j], w3[j].
struct NetBf16 {
    bf16 *w1t, *w2t, *w2, *w3;
};

__global__ __launch_bounds__(256) void k_mlp_prepare(const float *__restrict__ p, NetBf16 q) {
    for (int t = blockIdx.x * 256 + threadIdx.x; t < NH * NH; t += gridDim.x * 256) {
        const int i = t / NH, j = t % NH;
        const bf16 v = to_bf16(p[OFF_W2 + i * NH + j]);
        q.w2[i * NH + j] = v;
        q.w2t[j * NH + i] = v;
        if (i < NF) q.w1t[j * NF + i] = to_bf16(p[OFF_W1 + i * NH + j]);
        if (i == 0) q.w3[j] = to_bf16(p[OFF_W3 + j]);
    }
}

// Shared forward part of one 64-row tile.  On return: xs (bf16 inputs),
// h1 (bf16, row-major), z1 signs in m1, and per lane the layer-2 outputs
// h2 (bf16-rounded, as float) of its two 32 x 32 blocks plus their masks.
struct Lds {
    bf16 w1t[NH * PF];
    bf16 w2t[NH * PH];
    bf16 xs[ROWS * PF];
    bf16 h1[ROWS * PH];
    float part[ROWS][4];
};

// (16-byte pieces: eight loads per thread in flight instead of 64 two-byte ones)
__device__ inline void load_weights(Lds &L, const NetBf16 &q) {
    constexpr int N2 = NH * NH / 8 / 256;
    bf16x8 w[N2];
    for (int k = 0; k < N2; ++k) w[k] = ld8(q.w2t + 8 * (threadIdx.x + 256 * k));
    const bf16x8 w1 = ld8(q.w1t + 8 * threadIdx.x);  // NH * NF = 8 * 256
    for (int k = 0; k < N2; ++k) {
        const int t = 8 * (threadIdx.x + 256 * k);
        *reinterpret_cast<bf16x8 *>(&L.w2t[(t / NH) * PH + t % NH]) = w[k];
    }
    *reinterpret_cast<bf16x8 *>(&L.w1t[(threadIdx.x / 2) * PF + 8 * (threadIdx.x % 2)]) = w1;
}
static_assert(NH * NF == 8 * 256 && NH * NH % (8 * 256) == 0, "pieces of the weights");

// One tile's inputs: four features per thread, loaded ahead of the tile
// before (fetch) and rounded into LDS (put).
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // feat may be any float pointer
__device__ inline f32x4 fetch_tile(const float *__restrict__ X, int64_t row0, int64_t M) {
    if (M < 1) return f32x4{0.f, 0.f, 0.f, 0.f};
    const int64_t row = row0 + threadIdx.x / 4;
    const f32x4 v = *reinterpret_cast<const f32x4u *>(X + min(row, M - 1) * NF + 4 * (threadIdx.x % 4));
    return row < M ? v : f32x4{0.f, 0.f, 0.f, 0.f};
}
__device__ inline bf16x4 round4(const f32x4 &v) {
    return bf16x4{to_bf16(v[0]), to_bf16(v[1]), to_bf16(v[2]), to_bf16(v[3])};
}
__device__ inline void put_tile(Lds &L, const f32x4 &v) {
    *reinterpret_cast<bf16x4 *>(&L.xs[(threadIdx.x / 4) * PF + 4 * (threadIdx.x % 4)]) = round4(v);
}

// Wave w: row block rb = w >> 1, column blocks 2 (w & 1) + {0, 1}.
// With h1t, the hidden layer is also written transposed (pitch PR): the four
// consecutive rows a lane holds are one 8-byte store.
__device__ inline void forward_tile(Lds &L, const float *__restrict__ b1, const float *__restrict__ b2,
                                    f32x16 (&h2)[2], uint32_t (&mask2)[2], bf16 *h1t = nullptr) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rb = wave >> 1, hi = lane >> 5, lo = lane & 31;
    // layer 1: h1 = relu(x W1 + b1)
    for (int c = 0; c < 2; ++c) {
        const int cb = 2 * (wave & 1) + c;
        f32x16 acc = {};
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld8(&L.xs[(rb * 32 + lo) * PF + 8 * hi]),
                                                     ld8(&L.w1t[(cb * 32 + lo) * PF + 8 * hi]), acc, 0, 0, 0);
        const int col = cb * 32 + lo;
        const float bias = b1[col];
        for (int i = 0; i < 16; i += 4) {
            const int row = rb * 32 + 8 * (i >> 2) + 4 * hi;
            bf16x4 h;
            for (int e = 0; e < 4; ++e) {
                h[e] = to_bf16(fmaxf(acc[i + e] + bias, 0.0f));
                L.h1[(row + e) * PH + col] = h[e];
            }
            if (h1t) *reinterpret_cast<bf16x4 *>(&h1t[col * PR + row]) = h;
        }
    }
    __syncthreads();
    // layer 2: h2 = relu(h1 W2 + b2)
    for (int c = 0; c < 2; ++c) {
        const int cb = 2 * (wave & 1) + c;
        f32x16 acc = {};
        for (int kk = 0; kk < NH / 16; ++kk)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld8(&L.h1[(rb * 32 + lo) * PH + 16 * kk + 8 * hi]),
                                                         ld8(&L.w2t[(cb * 32 + lo) * PH + 16 * kk + 8 * hi]), acc,
                                                         0, 0, 0);
        const float bias = b2[cb * 32 + lo];
        uint32_t mk = 0;
        for (int i = 0; i < 16; ++i) {
            const float z = acc[i] + bias;
            mk |= (z > 0.0f ? 1u : 0u) << i;
            h2[c][i] = from_bf16(to_bf16(fmaxf(z, 0.0f)));
        }
        mask2[c] = mk;
    }
}

// Sums of sixteen values over the 32 lanes of a half-wave, each the same
// tree of additions as a butterfly over lane distances 1, 2, 4, 8, 16: each
// step adds the lane's half of the values to the partner's other half, so
// that 16 exchanges do what 80 would.  Returns, in lane l, the sum of value
// 8 b0 + 4 b1 + 2 b2 + b3 for the bits b of l (bit 4 of l: the same).
__device__ inline float half_sums(const float (&v)[16]) {
    const int lane = threadIdx.x;
    float a[8], b[4], c[2];
    for (int i = 0; i < 8; ++i) {
        const bool up = lane & 1;
        a[i] = (up ? v[8 + i] : v[i]) + __shfl_xor(up ? v[i] : v[8 + i], 1);
    }
    for (int i = 0; i < 4; ++i) {
        const bool up = lane & 2;
        b[i] = (up ? a[4 + i] : a[i]) + __shfl_xor(up ? a[i] : a[4 + i], 2);
    }
    for (int i = 0; i < 2; ++i) {
        const bool up = lane & 4;
        c[i] = (up ? b[2 + i] : b[i]) + __shfl_xor(up ? b[i] : b[2 + i], 4);
    }
    const bool up = lane & 8;
    const float d = (up ? c[1] : c[0]) + __shfl_xor(up ? c[0] : c[1], 8);
    return d + __shfl_xor(d, 16);
}

// ------------------------------------------------------------------ forward
__global__ __launch_bounds__(256) void k_mlp_fwd(const float *__restrict__ p, NetBf16 q, const float *__restrict__ X,
                                                 int64_t M, float *__restrict__ score) {
    __shared__ Lds L;
    load_weights(L, q);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rb = wave >> 1, hi = lane >> 5, lo = lane & 31;
    const int64_t ntiles = (M + ROWS - 1) / ROWS;
    float w3[2];
    for (int c = 0; c < 2; ++c) w3[c] = from_bf16(q.w3[(2 * (wave & 1) + c) * 32 + lo]);
    f32x4 x = fetch_tile(X, (int64_t)blockIdx.x * ROWS, M);
    for (int64_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        __syncthreads();
        put_tile(L, x);
        if (t + gridDim.x < ntiles) x = fetch_tile(X, (t + gridDim.x) * ROWS, M);
        __syncthreads();
        f32x16 h2[2];
        uint32_t mk[2];
        forward_tile(L, p + OFF_B1, p + OFF_B2, h2, mk);
        // layer 3: s = h2 W3 + b3 (deterministic: lanes, then blocks in order)
        for (int c = 0; c < 2; ++c) {
            float v[16];
            for (int i = 0; i < 16; ++i) v[i] = h2[c][i] * w3[c];
            const float sum = half_sums(v);
            if (lo < 16) {
                const int i = ((lo & 1) << 3) | ((lo & 2) << 1) | ((lo & 4) >> 1) | (lo >> 3);
                L.part[rb * 32 + 8 * (i >> 2) + 4 * hi + (i & 3)][2 * (wave & 1) + c] = sum;
            }
        }
        __syncthreads();
        if (threadIdx.x < ROWS) {
            const int64_t row = t * ROWS + threadIdx.x;
            const float *pp = L.part[threadIdx.x];
            if (row < M) score[row] = p[OFF_B3] + ((pp[0] + pp[1]) + (pp[2] + pp[3]));
        }
    }
}

// ------------------------------------------------------------------ loss
// Softmax cross-entropy with the probability mass of the winner set, per
// election e over rows [off[e], off[e+1]):
//   loss_e = log sum_all exp(s) - log sum_winners exp(s),
//   ds = (softmax over all - softmax over winners, on winners) / E.
// The sums go row a + lane, a + lane + 64, .. per lane of one wavefront, then
// over its lanes, whichever kernel runs: the results are the same bit for bit.
__device__ inline float wave_max(float v) {
    for (int o = 1; o < 64; o <<= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}
// one wavefront: ex(r) = exp(score[r] - max) summed over all rows and over the winners
template <typename F>
__device__ inline void wave_sums(const uint8_t *__restrict__ winner, int64_t a, int64_t b, F ex, float &sa, float &sw) {
    sa = sw = 0.f;
    for (int64_t r = a + (threadIdx.x & 63); r < b; r += 64) {
        const float x = ex(r);
        sa += x;
        if (winner[r]) sw += x;
    }
    for (int o = 1; o < 64; o <<= 1) {
        sa += __shfl_xor(sa, o);
        sw += __shfl_xor(sw, o);
    }
}
__device__ inline float row_grad(float x, bool winner, float sa, float sw, float inv_e) {
    const bool ok = sw > 0.f;
    float g = x / sa;
    if (winner && ok) g -= x / sw;
    return ok ? g * inv_e : 0.f;
}
__device__ inline float seg_loss(float sa, float sw) { return sw > 0.f ? logf(sa) - logf(sw) : 0.f; }

// Few elections: a workgroup each.  The exponentials of elections of up to
// SEG_KEEP rows are computed once, by all threads, into LDS, and the first
// wavefront adds them up.  With a wavefront doing all of it, 128 elections of
// 1150 rows left half the chip idle and took 25 us, of which this 7.
constexpr int SEG_KEEP = 8192;
__global__ __launch_bounds__(256) void k_seg_loss(const float *__restrict__ score, const int64_t *__restrict__ off,
                                                  const uint8_t *__restrict__ winner, int32_t E,
                                                  float *__restrict__ ds, float *__restrict__ loss) {
    __shared__ float ex[SEG_KEEP];
    __shared__ float red[4], sums[2];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t e = blockIdx.x;
    const int64_t a = off[e], b = off[e + 1];
    const bool keep = b - a <= SEG_KEEP;
    float mx = -INFINITY;
    for (int64_t r = a + threadIdx.x; r < b; r += 256) {
        const float s = score[r];
        if (keep) ex[r - a] = s;
        mx = fmaxf(mx, s);
    }
    mx = wave_max(mx);
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    if (keep)
        for (int64_t r = threadIdx.x; r < b - a; r += 256) ex[r] = expf(ex[r] - mx);
    __syncthreads();
    auto x_of = [&](int64_t r) { return keep ? ex[r - a] : expf(score[r] - mx); };
    if (wave == 0) {
        float sa, sw;
        wave_sums(winner, a, b, x_of, sa, sw);
        if (lane == 0) {
            sums[0] = sa;
            sums[1] = sw;
        }
    }
    __syncthreads();
    const float sa = sums[0], sw = sums[1], inv_e = 1.0f / (float)E;
    for (int64_t r = a + threadIdx.x; r < b; r += 256) ds[r] = row_grad(x_of(r), winner[r], sa, sw, inv_e);
    if (threadIdx.x == 0) loss[e] = seg_loss(sa, sw);
}

// Many elections: a wavefront each, no LDS.
__global__ __launch_bounds__(256) void k_seg_loss_many(const float *__restrict__ score,
                                                       const int64_t *__restrict__ off,
                                                       const uint8_t *__restrict__ winner, int32_t E,
                                                       float *__restrict__ ds, float *__restrict__ loss) {
    const int lane = threadIdx.x & 63;
    const int64_t e = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (e >= E) return;
    const int64_t a = off[e], b = off[e + 1];
    float mx = -INFINITY;
    for (int64_t r = a + lane; r < b; r += 64) mx = fmaxf(mx, score[r]);
    mx = wave_max(mx);
    auto x_of = [&](int64_t r) { return expf(score[r] - mx); };
    float sa, sw;
    wave_sums(winner, a, b, x_of, sa, sw);
    const float inv_e = 1.0f / (float)E;
    for (int64_t r = a + lane; r < b; r += 64) ds[r] = row_grad(x_of(r), winner[r], sa, sw, inv_e);
    if (lane == 0) loss[e] = seg_loss(sa, sw);
}

// ------------------------------------------------------------------ backward
// A share of the tiles (share s of n: tiles s, s + n, ..) has its
// parameter-gradient partials accumulated in registers, after the forward
// part is recomputed, and written once to partial[s][NPARAM].  The number of
// shares is fixed by the rows, not by the launch, so that the gradient is the
// same however many workgroups run (one per CU: the LDS holds no second).
// Bound by latency: four wavefronts per CU between barriers, so the next
// tile's inputs are loaded a tile ahead and the transposed operands are
// written as 8-byte stores of the four consecutive rows a lane holds.
struct BwdLds {
    Lds f;
    bf16 dz2[ROWS * PH];   // row-major
    bf16 dz2t[NH * PR];    // transposed
    bf16 h1t[NH * PR];     // transposed h1
    bf16 dz1t[NH * PR];    // transposed dz1
    bf16 xt[NF * PR];      // transposed inputs
    float ds[ROWS];
    float red[4][NH];
};

//
// With `step`, the train step's Adam counter is advanced here: the launch
// right before the one that uses it, so that a step which fails earlier leaves
// the counter where the parameters are.
__global__ __launch_bounds__(256) void k_mlp_bwd(const float *__restrict__ p, NetBf16 q, const float *__restrict__ X,
                                                 const float *__restrict__ dsg, int64_t M, int32_t shares,
                                                 float *__restrict__ partial, int32_t *__restrict__ step) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    BwdLds &L = *reinterpret_cast<BwdLds *>(smem);
    if (step && blockIdx.x == 0 && threadIdx.x == 0) step[0] += 1;
    load_weights(L.f, q);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int rb = wave >> 1, hi = lane >> 5, lo = lane & 31;
    // B operands of dh1 = dz2 W2^T stay in registers: W2[i][16 kk + 8 hi ..]
    bf16x8 w2f[2][NH / 16];
    for (int c = 0; c < 2; ++c)
        for (int kk = 0; kk < NH / 16; ++kk)
            w2f[c][kk] = ld8(&q.w2[(int64_t)((2 * (wave & 1) + c) * 32 + lo) * NH + 16 * kk + 8 * hi]);

    float w3c[2];
    for (int c = 0; c < 2; ++c) w3c[c] = from_bf16(q.w3[(2 * (wave & 1) + c) * 32 + lo]);

    const int64_t ntiles = (M + ROWS - 1) / ROWS;
    auto fetch_ds = [&](int64_t t) {
        const int64_t row = t * ROWS + threadIdx.x;
        return threadIdx.x < ROWS && row < M ? dsg[row] : 0.f;
    };
    for (int32_t share = blockIdx.x; share < shares; share += gridDim.x) {
    f32x16 gw2[4] = {};     // dW2 blocks (ib = wave, jb = 0..3)
    f32x4 gw1[2] = {};      // dW1 blocks (16 x 16): ib = 2 wave + {0,1}
    float gw3[2] = {0.f, 0.f}, gb2[2] = {0.f, 0.f}, gb1[2] = {0.f, 0.f}, gb3 = 0.f;
    f32x4 x = fetch_tile(X, (int64_t)share * ROWS, M);
    float dsv = fetch_ds(share);
    for (int64_t t = share; t < ntiles; t += shares) {
        __syncthreads();
        put_tile(L.f, x);
        {  // transposed inputs for dW1
            const bf16x4 r = round4(x);
            for (int e = 0; e < 4; ++e) L.xt[(4 * (threadIdx.x % 4) + e) * PR + threadIdx.x / 4] = r[e];
        }
        if (threadIdx.x < ROWS) L.ds[threadIdx.x] = dsv;
        if (t + shares < ntiles) {  // the next tile's rows, in flight during this one
            x = fetch_tile(X, (t + shares) * ROWS, M);
            dsv = fetch_ds(t + shares);
        }
        __syncthreads();
        f32x16 h2[2];
        uint32_t mk2[2];
        forward_tile(L.f, p + OFF_B1, p + OFF_B2, h2, mk2, L.h1t);
        // dz2 = mask2 * ds * w3; dW3 += h2 ds; db2 += dz2 (from the rounded dz2)
        for (int c = 0; c < 2; ++c) {
            const int cb = 2 * (wave & 1) + c;
            const int col = cb * 32 + lo;
            const float w3 = w3c[c];
            float s3 = 0.f, s2 = 0.f;
            for (int i = 0; i < 16; i += 4) {
                const int row = rb * 32 + 8 * (i >> 2) + 4 * hi;
                bf16x4 dz;
                for (int e = 0; e < 4; ++e) {
                    const float dsr = L.ds[row + e];
                    s3 += h2[c][i + e] * dsr;
                    dz[e] = to_bf16(((mk2[c] >> (i + e)) & 1u) ? dsr * w3 : 0.0f);
                    s2 += from_bf16(dz[e]);
                    L.dz2[(row + e) * PH + col] = dz[e];
                }
                *reinterpret_cast<bf16x4 *>(&L.dz2t[col * PR + row]) = dz;  // four consecutive rows
            }
            gw3[c] += s3;
            gb2[c] += s2;
        }
        if (threadIdx.x == 192) {  // (row order)
            float s = 0.f;
#pragma unroll 16
            for (int r = 0; r < ROWS; ++r) s += L.ds[r];
            gb3 += s;
        }
        __syncthreads();
        // dW2[i][j] += sum_rows h1[r][i] dz2[r][j]; wave owns i-block = wave
        for (int jb = 0; jb < 4; ++jb)
            for (int kk = 0; kk < ROWS / 16; ++kk)
                gw2[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    ld8(&L.h1t[(wave * 32 + lo) * PR + 16 * kk + 8 * hi]),
                    ld8(&L.dz2t[(jb * 32 + lo) * PR + 16 * kk + 8 * hi]), gw2[jb], 0, 0, 0);
        // dh1 = dz2 W2^T; dz1 = mask1 * dh1 (mask1 from h1 > 0)
        for (int c = 0; c < 2; ++c) {
            const int ib = 2 * (wave & 1) + c;
            f32x16 acc = {};
            for (int kk = 0; kk < NH / 16; ++kk)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ld8(&L.dz2[(rb * 32 + lo) * PH + 16 * kk + 8 * hi]),
                                                             w2f[c][kk], acc, 0, 0, 0);
            const int col = ib * 32 + lo;
            float s1 = 0.f;
            for (int i = 0; i < 16; i += 4) {
                const int row = rb * 32 + 8 * (i >> 2) + 4 * hi;
                const bf16x4 h = *reinterpret_cast<const bf16x4 *>(&L.h1t[col * PR + row]);
                bf16x4 dz;
                for (int e = 0; e < 4; ++e) {
                    dz[e] = to_bf16(from_bf16(h[e]) > 0.0f ? acc[i + e] : 0.0f);
                    s1 += from_bf16(dz[e]);
                }
                *reinterpret_cast<bf16x4 *>(&L.dz1t[col * PR + row]) = dz;
            }
            gb1[c] += s1;
        }
        __syncthreads();
        // dW1[f][i] += sum_rows x[r][f] dz1[r][i] (16 x 16 blocks, k = rows)
        for (int c = 0; c < 2; ++c) {
            const int ib = 2 * wave + c;
            for (int kk = 0; kk < ROWS / 32; ++kk)
                gw1[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    ld8(&L.xt[(lane & 15) * PR + 32 * kk + 8 * (lane >> 4)]),
                    ld8(&L.dz1t[(ib * 16 + (lane & 15)) * PR + 32 * kk + 8 * (lane >> 4)]), gw1[c], 0, 0, 0);
        }
    }
    // write this workgroup's partials (fixed order reductions only)
    float *out = partial + (int64_t)share * NPARAM;
    for (int jb = 0; jb < 4; ++jb)
        for (int i = 0; i < 16; ++i) {
            const int r = wave * 32 + 8 * (i >> 2) + 4 * hi + (i & 3);
            out[OFF_W2 + r * NH + jb * 32 + lo] = gw2[jb][i];
        }
    for (int c = 0; c < 2; ++c)
        for (int i = 0; i < 4; ++i) {
            const int f = 4 * (lane >> 4) + i;
            out[OFF_W1 + f * NH + (2 * wave + c) * 16 + (lane & 15)] = gw1[c][i];
        }
    // bias and W3 gradients: combine the two half-waves and the two row blocks
    __syncthreads();
    for (int c = 0; c < 2; ++c) {
        const int col = (2 * (wave & 1) + c) * 32 + lo;
        // slot: row block rb, half hi -> red[2 rb + hi][col]
        L.red[2 * rb + hi][col] = gw3[c];
    }
    __syncthreads();
    if (threadIdx.x < NH) {
        const int col = threadIdx.x;
        out[OFF_W3 + col] = (L.red[0][col] + L.red[1][col]) + (L.red[2][col] + L.red[3][col]);
    }
    __syncthreads();
    for (int c = 0; c < 2; ++c) L.red[2 * rb + hi][(2 * (wave & 1) + c) * 32 + lo] = gb2[c];
    __syncthreads();
    if (threadIdx.x < NH) {
        const int col = threadIdx.x;
        out[OFF_B2 + col] = (L.red[0][col] + L.red[1][col]) + (L.red[2][col] + L.red[3][col]);
    }
    __syncthreads();
    for (int c = 0; c < 2; ++c) L.red[2 * rb + hi][(2 * (wave & 1) + c) * 32 + lo] = gb1[c];
    __syncthreads();
    if (threadIdx.x < NH) {
        const int col = threadIdx.x;
        out[OFF_B1 + col] = (L.red[0][col] + L.red[1][col]) + (L.red[2][col] + L.red[3][col]);
    }
    if (threadIdx.x == 192) out[OFF_B3] = gb3;
    }
}

// Adam (FP32 master weights), bias-corrected, step t >= 1.
struct AdamArgs {
    float *p, *m1, *m2;
    float lr, b1, b2, eps;
    int32_t t_host;
    int32_t *t_dev;  // when given, the device counter (the train step's backward advances it)
};
__device__ inline void adam_step(const AdamArgs &a, int k, float gk) {
    const int32_t t = a.t_dev ? *a.t_dev : a.t_host;
    const float m = a.b1 * a.m1[k] + (1.f - a.b1) * gk;
    const float v = a.b2 * a.m2[k] + (1.f - a.b2) * gk * gk;
    a.m1[k] = m;
    a.m2[k] = v;
    const float ah = m / (1.f - powf(a.b1, (float)t));
    const float vh = v / (1.f - powf(a.b2, (float)t));
    a.p[k] -= a.lr * ah / (sqrtf(vh) + a.eps);
}
__global__ __launch_bounds__(256) void k_adam(AdamArgs a, const float *__restrict__ g) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < NPARAM) adam_step(a, k, g[k]);
}

// grad[k] = sum over shares of partial[share][k], in share order; with a.p,
// the parameter's Adam step follows.  One wavefront per 64 parameters, so
// that the additions, one after the other, spread over the whole chip with
// 64 loads in flight per thread (256 parameters per workgroup and few loads
// in flight took 122 us of a 292 us train step).
__global__ __launch_bounds__(64) void k_mlp_reduce(const float *__restrict__ partial, int32_t shares,
                                                   float *__restrict__ grad, AdamArgs a) {
    constexpr int FLY = 64;
    const int k = blockIdx.x * 64 + threadIdx.x;
    if (k >= NPARAM) return;
    float s = 0.f;
    int b = 0;
    for (; b + FLY <= shares; b += FLY) {
        float v[FLY];
#pragma unroll
        for (int u = 0; u < FLY; ++u) v[u] = partial[(int64_t)(b + u) * NPARAM + k];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < FLY; ++u) s += v[u];
    }
#pragma unroll 8
    for (; b < shares; ++b) s += partial[(int64_t)b * NPARAM + k];
    grad[k] = s;
    if (a.p) adam_step(a, k, s);
}

size_t bwd_lds_bytes() { return sizeof(BwdLds); }

constexpr size_t W2_BYTES = sizeof(bf16) * NH * NH, W1_BYTES = sizeof(bf16) * NH * NF;
constexpr size_t PREPARED_BYTES = 2 * W2_BYTES + W1_BYTES + 256 + 256;

int prepare(schulze_ctx *ctx, hipStream_t s, const float *params, NetBf16 &q) {
    int rc = ws_reserve(ctx, WS_MLP, PREPARED_BYTES);
    if (rc != SCHULZE_OK) return rc;
    char *b = static_cast<char *>(ctx->ws[WS_MLP]);
    q.w2t = reinterpret_cast<bf16 *>(b);
    q.w2 = reinterpret_cast<bf16 *>(b + W2_BYTES);
    q.w1t = reinterpret_cast<bf16 *>(b + 2 * W2_BYTES);
    q.w3 = reinterpret_cast<bf16 *>(b + 2 * W2_BYTES + W1_BYTES + 256);
    SCHULZE_LAUNCH(ctx, K_MLP_PREP, s, k_mlp_prepare<<<dim3(16), dim3(256), 0, s>>>(params, q));
    return SCHULZE_OK;
}

int grid_for(schulze_ctx *ctx, int64_t M) {
    int64_t g = std::min<int64_t>((M + ROWS - 1) / ROWS, (int64_t)ctx->num_cus * 2);
    return (int)std::max<int64_t>(g, 1);
}

}  // namespace

extern "C" int schulze_mlp_forward(schulze_ctx *ctx, void *stream, const float *params, const float *feat, int64_t M,
                                   float *score) {
    if (!ctx || !params || !feat || !score || M < 0) return SCHULZE_EINVAL;
    if (bind_device(ctx) != SCHULZE_OK) return SCHULZE_EDEVICE;
    if (M == 0) return SCHULZE_OK;
    hipStream_t s = (hipStream_t)stream;
    NetBf16 q;
    int rc = prepare(ctx, s, params, q);
    if (rc != SCHULZE_OK) return rc;
    SCHULZE_LAUNCH(ctx, K_MLP_FWD, s,
                   k_mlp_fwd<<<dim3((unsigned)grid_for(ctx, M)), dim3(256), 0, s>>>(params, q, feat, M, score));
    return SCHULZE_OK;
}

namespace {

// A workgroup per election while all of them stay resident together (four per
// CU by their LDS), a wavefront each beyond.  The lengths of the elections are
// on the device, so the rule knows their number only.
int loss_of(schulze_ctx *ctx, hipStream_t s, const float *score, const int64_t *offsets, const uint8_t *winner,
            int32_t E, float *dscore, float *loss) {
    if (E <= 4 * ctx->num_cus)
        SCHULZE_LAUNCH(ctx, K_MLP_LOSS, s,
                       k_seg_loss<<<dim3((unsigned)E), dim3(256), 0, s>>>(score, offsets, winner, E, dscore, loss));
    else
        SCHULZE_LAUNCH(ctx, K_MLP_LOSS, s,
                       k_seg_loss_many<<<dim3((unsigned)ceil_div(E, 4)), dim3(256), 0, s>>>(score, offsets, winner, E,
                                                                                          dscore, loss));
    return SCHULZE_OK;
}

// What a backward over M rows needs besides its launches, before anything is
// queued: a call that fails here has changed nothing.
int backward_reserve(schulze_ctx *ctx, int64_t M) {
    int rc = ws_reserve(ctx, WS_MLP, PREPARED_BYTES);
    if (rc != SCHULZE_OK) return rc;
    if ((rc = ws_reserve(ctx, WS_MLP_PARTIAL, sizeof(float) * (size_t)grid_for(ctx, M) * NPARAM)) != SCHULZE_OK)
        return rc;
    if (hipFuncSetAttribute((const void *)k_mlp_bwd, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)bwd_lds_bytes()) != hipSuccess)
        return SCHULZE_EDEVICE;
    return SCHULZE_OK;
}

// Backward of the prepared network (q) into grad, and its Adam step if
// adam.p is given (adam.t_dev, if given, is advanced first); arguments
// checked and backward_reserve done.
int backward(schulze_ctx *ctx, hipStream_t s, const float *params, const NetBf16 &q, const float *feat, int64_t M,
             const float *dscore, float *grad, const AdamArgs &adam) {
    const int shares = grid_for(ctx, M);
    const int G = std::min(shares, ctx->num_cus);
    float *partial = static_cast<float *>(ctx->ws[WS_MLP_PARTIAL]);
    SCHULZE_LAUNCH(ctx, K_MLP_BWD, s,
                   k_mlp_bwd<<<dim3((unsigned)G), dim3(256), bwd_lds_bytes(), s>>>(params, q, feat, dscore, M, shares,
                                                                                  partial, adam.t_dev));
    SCHULZE_LAUNCH(ctx, K_MLP_BWD, s,
                   k_mlp_reduce<<<dim3((unsigned)ceil_div(NPARAM, 64)), dim3(64), 0, s>>>(partial, shares, grad, adam));
    return SCHULZE_OK;
}

}  // namespace

extern "C" int schulze_mlp_backward(schulze_ctx *ctx, void *stream, const float *params, const float *feat, int64_t M,
                                    const float *dscore, float *grad) {
    if (!ctx || !params || !feat || !dscore || !grad || M < 0) return SCHULZE_EINVAL;
    if (bind_device(ctx) != SCHULZE_OK) return SCHULZE_EDEVICE;
    hipStream_t s = (hipStream_t)stream;
    NetBf16 q;
    int rc = backward_reserve(ctx, M);
    if (rc != SCHULZE_OK || (rc = prepare(ctx, s, params, q)) != SCHULZE_OK) return rc;
    return backward(ctx, s, params, q, feat, M, dscore, grad, AdamArgs{});
}

extern "C" int schulze_mlp_loss(schulze_ctx *ctx, void *stream, const float *score, const int64_t *offsets,
                                const uint8_t *winner, int32_t E, float *dscore, float *loss) {
    if (!ctx || !score || !offsets || !winner || !dscore || !loss || E < 1) return SCHULZE_EINVAL;
    if (bind_device(ctx) != SCHULZE_OK) return SCHULZE_EDEVICE;
    hipStream_t s = (hipStream_t)stream;
    return loss_of(ctx, s, score, offsets, winner, E, dscore, loss);
}

extern "C" int schulze_mlp_adam(schulze_ctx *ctx, void *stream, float *params, const float *grad, float *adam_m,
                                float *adam_v, float lr, float beta1, float beta2, float eps, int32_t step) {
    if (!ctx || !params || !grad || !adam_m || !adam_v || step < 1) return SCHULZE_EINVAL;
    if (bind_device(ctx) != SCHULZE_OK) return SCHULZE_EDEVICE;
    hipStream_t s = (hipStream_t)stream;
    SCHULZE_LAUNCH(ctx, K_MLP_ADAM, s,
                   k_adam<<<dim3((unsigned)ceil_div(NPARAM, 256)), dim3(256), 0, s>>>(
                       AdamArgs{params, adam_m, adam_v, lr, beta1, beta2, eps, step, nullptr}, grad));
    return SCHULZE_OK;
}

extern "C" int schulze_mlp_train_step(schulze_ctx *ctx, void *stream, const schulze_mlp *net,
                                      const schulze_train_batch *b, float *loss) {
    if (!ctx || !net || !b || !loss) return SCHULZE_EINVAL;
    if (!net->params || !net->adam_m || !net->adam_v || !net->grad || !net->step) return SCHULZE_EINVAL;
    if (!b->feat || !b->offsets || !b->winner || b->M < 1 || b->E < 1) return SCHULZE_EINVAL;
    if (!(net->lr > 0.f) || !(net->beta1 >= 0.f && net->beta1 < 1.f) || !(net->beta2 >= 0.f && net->beta2 < 1.f) ||
        !(net->eps > 0.f))
        return SCHULZE_EINVAL;
    if (bind_device(ctx) != SCHULZE_OK) return SCHULZE_EDEVICE;
    hipStream_t s = (hipStream_t)stream;
    // scores and their gradient live in the workspace
    const size_t vec = round_up(sizeof(float) * (size_t)b->M, 256);
    int rc = ws_reserve(ctx, WS_MLP_TRAIN, 2 * vec);
    if (rc != SCHULZE_OK || (rc = backward_reserve(ctx, b->M)) != SCHULZE_OK) return rc;
    float *score = static_cast<float *>(ctx->ws[WS_MLP_TRAIN]);
    float *dscore = reinterpret_cast<float *>(static_cast<char *>(ctx->ws[WS_MLP_TRAIN]) + vec);
    NetBf16 q;
    if ((rc = prepare(ctx, s, net->params, q)) != SCHULZE_OK) return rc;
    SCHULZE_LAUNCH(ctx, K_MLP_FWD, s,
                   k_mlp_fwd<<<dim3((unsigned)grid_for(ctx, b->M)), dim3(256), 0, s>>>(net->params, q, b->feat, b->M,
                                                                                       score));
    if ((rc = loss_of(ctx, s, score, b->offsets, b->winner, b->E, dscore, loss)) != SCHULZE_OK) return rc;
    return backward(ctx, s, net->params, q, b->feat, b->M, dscore, net->grad,
                    AdamArgs{net->params, net->adam_m, net->adam_v, net->lr, net->beta1, net->beta2, net->eps, 0,
                             net->step});
}

extern "C" int schulze_mlp_param_count(void) { return NPARAM; }
