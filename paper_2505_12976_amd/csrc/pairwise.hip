// Pairwise preference counts d[x][y] (Section 2.1: profile of weak orders).
//
// d[x][y] is the total weight of voters who list x and list y later or not
// at all.  Ballots are split by a scan into full rankings (at least m-1
// listed candidates) and truncated ballots, which take different routes:
//
//  * Bit-plane counting.  The ranks of 32 voters are kept as bit planes, one
//    32-bit word per candidate and bit (a bit per voter).  For one (x, y)
//    pair the mask of the voters with pos(x) < pos(y) comes from the bits
//    from the lowest up: lt = (~x & y) | (~(x ^ y) & lt), one v_bitop3_b32
//    per bit, and one v_bcnt_u32_b32 adds its population count: (bits + 1)
//    instructions for 32 comparisons, where a packed subtraction and a dot
//    product took 32.  Voter weights go through the same masks, bit plane by
//    bit plane of the weights.
//    - Full rankings have no ties, so only tiles with x-block <= y-block are
//      counted and d[y][x] = voters - d[x][y].
//    - Truncated ballots are counted the same way over the candidates U that
//      any truncated ballot lists (unlisted candidates share one sentinel
//      position, all ones, so ties count for neither side), over all ordered
//      tiles.  One extra always-sentinel column gives R[x], the number of
//      truncated ballots listing x, and d[x][y] = R[x] for x in U, y outside
//      U.
//  * Pair scattering, for truncated ballots when U is large: d[x][y] =
//    R[x] - C[y][x], where C[y][x] is the weight of ballots listing y before
//    x; the listed pairs are scattered with atomics.
// A small decision kernel picks the cheaper truncated route on the device.
// Everything accumulates into one m x m uint32 matrix that a final pass
// completes and converts to the output dtype.
#include "internal.h"
#include "planes.h"
#include "row_pieces.h"
#include "tile_io.h"

namespace {

constexpr int CT = 128;           // count tile (candidates per side)
constexpr int COUNT_PER_CU = 3;   // workgroups of the count per CU (168 vector registers)
constexpr int MAX_BITS = 16;      // bit planes of a rank (m <= 65535)
constexpr int LONG_CHUNK = 256;   // ballots per list of the long-row scan
constexpr int SHORT_PER_WAVE = 8; // steps (groups of ballots) per wavefront of the short-row scan
constexpr int NPART = 64;         // partial sums of the pair-scattering cost

enum { MODE_SPARSE = 0, MODE_DENSE_U = 1 };

#define CNT_LDS __attribute__((address_space(3)))

// Workspace views (WS_BALLOT_META).
struct Meta {
    int32_t *ctr;            // [0] full rankings [1] truncated ballots [2] route
                             // [3] |U| [4] U-space pitch [6] longest truncated
                             // ballot [7] voter weights or-ed together [8] total
                             // weight of the full rankings (mod 2^32) [9] error of a
                             // repeated id (one-pass count) [32..33] total
                             // voter weight (64 bits) [34] its workgroups done
    unsigned long long *k2;  // NPART partial sums of k(k-1)/2 over truncated ballots
    int32_t *len;            // listed length per ballot
    int32_t *full_src;       // slot -> ballot of a full ranking
    int32_t *trunc_src;      // slot -> ballot of a truncated ballot
    uint8_t *in_u;           // candidate listed by some truncated ballot
    int32_t *ulist;          // U-space index -> candidate
    int32_t *umap;           // candidate -> U-space index or -1
};

// Ballot entry idx, -1 for padding.  The id type is a template parameter:
// a branch on it at every load made each load wait for the one before.
template <bool I32>
__device__ inline uint32_t load_raw(const void *ballots, int64_t idx) {
    if constexpr (I32)
        return static_cast<const uint32_t *>(ballots)[idx];
    else
        return static_cast<const uint16_t *>(ballots)[idx];
}
template <bool I32>
__device__ inline int32_t raw_id(uint32_t raw) {
    if constexpr (I32)
        return (int32_t)raw < 0 ? -1 : (int32_t)raw;
    else
        return raw == 0xFFFFu ? -1 : (int32_t)raw;
}
template <bool I32>
__device__ inline int32_t read_id(const void *ballots, int64_t idx) {
    return raw_id<I32>(load_raw<I32>(ballots, idx));
}

// ------------------------------------------------------------------ scan
// Listed length, id range check, full/truncated split (slots reserved once
// per workgroup: every reservation is an atomic on the same two counters,
// about 30 ns each one after the other, which with a reservation per 32
// ballots was most of the scan's time), candidates listed by truncated
// ballots, and the pair count of the truncated ballots.
__device__ inline void record_ballots(Meta meta, int nf, const int32_t *lf, int nt, const int32_t *lt) {
    __shared__ int32_t base_f, base_t;
    if (threadIdx.x == 0) {
        base_f = nf ? atomicAdd(&meta.ctr[0], nf) : 0;
        base_t = nt ? atomicAdd(&meta.ctr[1], nt) : 0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nf; i += blockDim.x) meta.full_src[base_f + i] = lf[i];
    for (int i = threadIdx.x; i < nt; i += blockDim.x) meta.trunc_src[base_t + i] = lt[i];
}

// Long rows: one wavefront per ballot, a workgroup of 16 takes `chunk`
// ballots (at most one workgroup per CU, so that there are few
// reservations), LONG_CHUNK to a list.  Bound by reading the ballots once:
// eight 16-byte pieces per lane in flight, and a piece whose ids are all
// below m takes one comparison; only ballots that end early are read again,
// as far as they go, to mark what they list.
template <bool I32>
__global__ __launch_bounds__(1024) void k_scan_long(const void *__restrict__ ballots, int64_t n, int32_t L, int32_t m,
                                                   int32_t chunk, Meta meta, int32_t *err) {
    using P = RowPieces<I32, true>;
    constexpr int FLY = 8;
    __shared__ int32_t lf[LONG_CHUNK], lt[LONG_CHUNK];
    __shared__ uint8_t kind[LONG_CHUNK];  // 0 none, 1 full, 2 truncated
    __shared__ int32_t nf, nt;
    // candidates listed by this workgroup's truncated ballots (m <= 65535):
    // byte stores of every workgroup to the same few lines were slower
    __shared__ uint32_t seen[65536 / 32];
    for (int32_t w = threadIdx.x; w < (m + 31) / 32; w += 1024) seen[w] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t c0 = (int64_t)blockIdx.x * chunk, c1 = min(n, c0 + chunk);
    bool bad = false;
    unsigned long long k2 = 0;
    int32_t longest = 0;  // listed by a truncated ballot
    for (int64_t v0 = c0; v0 < c1; v0 += LONG_CHUNK) {
        const int32_t here = (int32_t)min((int64_t)LONG_CHUNK, c1 - v0);
        for (int q = wave; q < here; q += 16) {
            const int64_t v = v0 + q;
            const P row(ballots, n, L, v);
            int32_t first = L, wrong = L;  // first padding entry, first id out of range
            for (int32_t j0 = 0; j0 < row.count; j0 += 64 * FLY) {
                v4u x[FLY];
                row.template load<FLY>(x, j0 + lane);
                for (int u = 0; u < FLY; ++u) {
                    const int32_t j = j0 + 64 * u + lane;
                    if (j >= row.count || P::top(x[u]) < (uint32_t)m) continue;
                    row.each(x[u], j, L, [&](int32_t t, uint32_t raw) {
                        const int32_t id = raw_id<I32>(raw);
                        if (id < 0)
                            first = min(first, t);
                        else if (id >= m)
                            wrong = min(wrong, t);
                    });
                }
                if (__ballot(first < L)) break;
            }
            for (int off = 32; off >= 1; off >>= 1) first = min(first, __shfl_xor(first, off));
            const int32_t k = first;
            bad |= wrong < k;
            const bool trunc = k < m - 1;
            if (trunc)
                for (int32_t j = lane; j < row.count && j * P::PER - row.head < k; j += 64) {
                    v4u x[1];
                    row.template load<1>(x, j);
                    row.each(x[0], j, k, [&](int32_t, uint32_t raw) {
                        const uint32_t bit = 1u << (raw & 31);
                        if (raw < (uint32_t)m && !(seen[raw >> 5] & bit)) atomicOr(&seen[raw >> 5], bit);
                    });
                }
            if (lane == 0) {
                meta.len[v] = k;
                kind[q] = trunc ? 2 : 1;
                if (trunc) {
                    k2 += (unsigned long long)k * (k - 1) / 2;
                    longest = max(longest, k);
                }
            }
        }
        __syncthreads();
        if (wave == 0) {  // the lists, in ballot order
            int32_t a = 0, b = 0;
            for (int q0 = 0; q0 < here; q0 += 64) {
                const int q = q0 + lane, kq = q < here ? kind[q] : 0;
                const uint64_t f = __ballot(kq == 1), t = __ballot(kq == 2), below = (1ull << lane) - 1ull;
                if (kq == 1) lf[a + __popcll(f & below)] = (int32_t)(v0 + q);
                if (kq == 2) lt[b + __popcll(t & below)] = (int32_t)(v0 + q);
                a += __popcll(f);
                b += __popcll(t);
            }
            if (lane == 0) {
                nf = a;
                nt = b;
            }
        }
        __syncthreads();
        record_ballots(meta, nf, lf, nt, lt);
        __syncthreads();  // the lists are copied
    }
    for (int32_t c = threadIdx.x; c < m; c += 1024)
        if ((seen[c >> 5] >> (c & 31)) & 1u) meta.in_u[c] = 1;
    if (bad) set_device_error(err, SCHULZE_EBALLOT);
    if (lane == 0 && k2) atomicAdd(&meta.k2[(blockIdx.x * 16 + wave) % NPART], k2);
    if (lane == 0 && longest > __hip_atomic_load(&meta.ctr[6], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(&meta.ctr[6], longest);
}

// Short rows (L <= 64): a wavefront takes 64 / L ballots at once (at most
// SHORT_BPW), one lane per entry, SHORT_PER_WAVE such steps with all their
// loads issued first, `rounds` times; a ballot's listed length is the
// first padding lane of its group (a wavefront ballot).  (More ballots per
// workgroup mean fewer list reservations on the two shared counters.)
constexpr int SHORT_BPW = 4;
constexpr int SHORT_ROUNDS = 4, SHORT_MAX_ROUNDS = 16;
template <bool I32>
__global__ __launch_bounds__(256) void k_scan_short(const void *__restrict__ ballots, int64_t n, int32_t L,
                                                    int32_t m, int32_t rounds, Meta meta, int32_t *err) {
    constexpr int PER_WG = 4 * SHORT_PER_WAVE * SHORT_BPW * SHORT_MAX_ROUNDS;
    __shared__ int32_t lf[PER_WG], lt[PER_WG];
    __shared__ int32_t nf, nt;
    // candidates listed by this workgroup's truncated ballots, as bits
    // (m <= 65535): one store per candidate and workgroup at the end instead
    // of a read of in_u at every entry, which made each step wait for memory
    __shared__ uint32_t seen[65536 / 32];
    if (threadIdx.x == 0) nf = nt = 0;
    for (int32_t w = threadIdx.x; w < (m + 31) / 32; w += 256) seen[w] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t bpw = min(SHORT_BPW, 64 / L);
    const int32_t sub = lane / L, t = lane - sub * L;
    const bool lane_ok = sub < bpw;
    const uint64_t group_bits = (L == 64) ? ~0ull : ((1ull << L) - 1ull);
    bool bad = false;
    unsigned long long k2 = 0;
    for (int round = 0; round < rounds; ++round) {
        const int64_t v0 = (((int64_t)blockIdx.x * rounds + round) * 4 + wave) * SHORT_PER_WAVE * bpw;
        int32_t c[SHORT_PER_WAVE];
        for (int q = 0; q < SHORT_PER_WAVE; ++q) {  // every load first
            const int64_t v = v0 + (int64_t)q * bpw + sub;
            // (every lane loads: a load under a condition is waited for inside it)
            c[q] = (int32_t)load_raw<I32>(ballots, lane_ok && v < n ? v * L + t : 0);
        }
        for (int q = 0; q < SHORT_PER_WAVE; ++q) {
            const int64_t v = v0 + (int64_t)q * bpw + sub;
            c[q] = lane_ok && v < n ? raw_id<I32>((uint32_t)c[q]) : -2;
        }
        for (int q = 0; q < SHORT_PER_WAVE; ++q) {
            const int64_t v = v0 + (int64_t)q * bpw + sub;
            const uint64_t pad = __ballot(c[q] < 0);  // -1 padding, -2 no ballot
            const uint64_t mine = lane_ok ? (pad >> (sub * L)) & group_bits : group_bits;
            const int k = mine ? (int)__builtin_ctzll(mine) : L;
            const bool live = lane_ok && v < n;
            const bool trunc = k < m - 1;
            if (live && t < k) {
                if (c[q] >= m) {
                    bad = true;
                } else if (trunc) {
                    const uint32_t bit = 1u << (c[q] & 31);
                    if (!(seen[c[q] >> 5] & bit)) atomicOr(&seen[c[q] >> 5], bit);
                }
            }
            if (live && t == 0) {
                meta.len[v] = k;
                if (trunc) {
                    lt[atomicAdd(&nt, 1)] = (int32_t)v;
                    k2 += (unsigned long long)k * (k - 1) / 2;
                } else {
                    lf[atomicAdd(&nf, 1)] = (int32_t)v;
                }
            }
        }
    }
    if (__ballot(bad) && lane == 0) set_device_error(err, SCHULZE_EBALLOT);
    for (int off = 32; off >= 1; off >>= 1) k2 += __shfl_xor(k2, off);
    if (lane == 0 && k2) atomicAdd(&meta.k2[(blockIdx.x * 4 + wave) % NPART], k2);
    __syncthreads();
    for (int32_t c = threadIdx.x; c < m; c += 256)
        if ((seen[c >> 5] >> (c & 31)) & 1u) meta.in_u[c] = 1;
    record_ballots(meta, nf, lf, nt, lt);
}

// ------------------------------------------------------------------ route decision
// One workgroup: U-space compaction (prefix sum over candidates) and the
// choice between the dense route over U and pair scattering for truncated
// ballots, by the time each is expected to take (picoseconds, from measured
// rates on MI355X): dense, the masks' instructions over the tiles at 45 T
// lane operations/s and the m x m accumulator written, read and converted;
// pair scattering, a pair's share of the bucketed accumulation or a
// device-wide atomic, and d written once; both have their own passes over the
// ballots (about 60 us).  The share is what a pair took when an item's row
// was found by a search (5-6 ps); the accumulation takes 2.4 ps at n = 10^6
// top-20 and 2.7 ps at n = 15553 top-150, so close to the border the dense
// route still runs where pairs would be faster.
constexpr double DENSE_RATE = 45.0;            // lane operations per picosecond
constexpr double ATOMIC_PAIR_COST = 66.0;
constexpr double BUCKETED_PAIR_COST = 6.0;

constexpr int ROUTE_THREADS = 1024;
constexpr int ROUTE_VEC = 4;  // 16-byte groups of flags per thread
static_assert(ROUTE_THREADS * 16 * ROUTE_VEC >= 65536, "every candidate's flag");
__global__ __launch_bounds__(ROUTE_THREADS) void k_route(int32_t m, int32_t short_L, Meta meta,
                                                         int64_t cap_words, double pair_cost) {
    __shared__ int32_t part[ROUTE_THREADS];
    // A thread takes consecutive flags (0 or 1 bytes; zero past m up to the
    // next 16 bytes), as ROUTE_VEC 16-byte loads issued together (a byte at
    // a time waited for memory at every flag).
    const int32_t groups = (m + 15) / 16;
    const int32_t gper = (groups + ROUTE_THREADS - 1) / ROUTE_THREADS;
    const int32_t g0 = (int32_t)threadIdx.x * gper;
    uint4 f[ROUTE_VEC];
    int32_t cnt = 0;
    const uint4 *in4 = reinterpret_cast<const uint4 *>(meta.in_u);
    for (int k = 0; k < ROUTE_VEC; ++k) f[k] = in4[k < gper && g0 + k < groups ? g0 + k : 0];
    for (int k = 0; k < ROUTE_VEC; ++k) {
        if (!(k < gper && g0 + k < groups)) f[k] = make_uint4(0u, 0u, 0u, 0u);
        cnt += __popc(f[k].x) + __popc(f[k].y) + __popc(f[k].z) + __popc(f[k].w);
    }
    part[threadIdx.x] = cnt;
    __syncthreads();
    for (int off = 1; off < ROUTE_THREADS; off <<= 1) {  // inclusive scan
        const int32_t add = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    int32_t idx = part[threadIdx.x] - cnt;
    auto place = [&](int32_t c, bool in) {
        if (in) {
            meta.ulist[idx] = c;
            meta.umap[c] = idx++;
        } else {
            meta.umap[c] = -1;
        }
    };
    for (int k = 0; k < ROUTE_VEC; ++k) {
        const uint32_t w[4] = {f[k].x, f[k].y, f[k].z, f[k].w};
        for (int e = 0; e < 16; ++e) {
            const int32_t c = 16 * (g0 + k) + e;
            if (k < gper && c < m) place(c, (w[e >> 2] >> (8 * (e & 3))) & 1u);
        }
    }
    if (threadIdx.x == 0) {
        const int32_t nu = part[ROUTE_THREADS - 1];
        const int32_t pitch = (nu + 1 + CT - 1) / CT * CT;  // room for one sentinel column
        const int64_t n_t = meta.ctr[1];
        unsigned long long k2 = 0;
        for (int i = 0; i < NPART; ++i) k2 += meta.k2[i];
        const int64_t groups = (n_t + 31) / 32;
        if (short_L) meta.ctr[6] = short_L;  // (the short-row scan does not look for the longest ballot)
        const int32_t bits = rank_bits(meta.ctr[6]);
        const double mm = (double)m * m;
        const double dense =
            (double)groups * (double)pitch * (double)pitch * (bits + 2) / DENSE_RATE + 3.0 * mm;
        const bool fits = groups * (int64_t)pitch * bits <= cap_words;
        const bool use_dense = fits && n_t > 0 && dense <= pair_cost * (double)k2 + mm;
        meta.ctr[2] = use_dense ? MODE_DENSE_U : MODE_SPARSE;
        meta.ctr[3] = nu;
        meta.ctr[4] = pitch;
    }
}

// ------------------------------------------------------------------ rank planes
// Group g of 32 voters (slots 32 g ..) as bit planes: word (g, b, c) holds
// bit b of candidate c's rank for every voter of the group, voter 2p + h at
// bit 16 h + p.  A workgroup scatters the ranks of one group over CH columns
// into LDS, two voters per 32-bit word, and each thread then transposes the
// 16 words of a column as two 16 x 16 bit matrices (four butterfly stages).
// Unlisted candidates keep all ones; slots past the last voter are zero in
// every column and count for no pair.  Every ballot lists distinct candidates
// iff together they set as many columns as they have entries (no ballot can
// set more).  With voter weights, the group's weights are kept as 32 bit
// planes too, and those of full rankings are summed.
struct PlaneArgs {
    const void *ballots;
    int32_t L, m;
    int32_t pitch, bits;  // full rankings; truncated ballots take theirs from meta
    Meta meta;
    const uint32_t *weight;  // nullptr: every voter counts once
    uint32_t *planes;
    uint32_t *wplanes;  // WEIGHT_WORDS per group
    int32_t *err;
    int64_t n;           // ballots of the profile
};

// The columns of a group in LDS (16 words each, CH apart) as planes at `out`;
// returns minus the ranks set in the thread's columns below `real`.
template <int CH, int THREADS>
__device__ inline int32_t planes_out(const uint32_t *buf, int32_t cn, int32_t real, uint32_t voters, int32_t bits,
                                     int64_t pitch, uint32_t *out) {
    int32_t extra = 0;
    for (int32_t c = threadIdx.x; c < cn; c += THREADS) {
        uint32_t w[16];
        for (int p = 0; p < 16; ++p) w[p] = buf[p * CH + c];
        transpose16(w);
        uint32_t unset = w[0];
        for (int b = 1; b < 16; ++b) unset &= w[b];
        if (c < real) extra -= __popc(voters & ~unset);
#pragma unroll
        for (int b = 0; b < MAX_BITS; ++b)
            if (b < bits) out[b * pitch + c] = w[b];
    }
    return extra;
}

// extra: entries placed less columns set, by thread; not zero in total if a
// ballot lists a candidate twice.  *total is zero on entry.
__device__ inline void check_repeats(int32_t extra, int32_t *total, int32_t *err) {
    for (int off = 32; off >= 1; off >>= 1) extra += __shfl_xor(extra, off);
    if ((threadIdx.x & 63) == 0 && extra) atomicAdd(total, extra);
    __syncthreads();
    if (threadIdx.x == 0 && *total != 0) set_device_error(err, SCHULZE_EBALLOT);
}

// One wavefront: the weights of a group's voters (lanes 0 .. 31 hold the voter
// of their bit, the others 0) as 32 bit planes and as 32 words of digits: word
// 4 p + j has the p-th four bits of the weights of the voters 4 i + j, i = 0 ..
// 7.  Returns the weights' sum.
constexpr int WEIGHT_WORDS = 64;
__device__ inline uint32_t weight_planes(uint32_t w, uint32_t *out) {
    const int lane = threadIdx.x & 63;
    uint32_t mine = 0u, sum = w, digits = 0u;
    for (int j = 0; j < 32; ++j) {
        const uint32_t mask = (uint32_t)__ballot((w >> j) & 1u);
        if (lane == j) mine = mask;
    }
    for (int i = 0; i < 8; ++i) digits |= ((__shfl(w, 4 * i + (lane & 3)) >> (lane & 28)) & 15u) << (4 * i);
    for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
    if (lane < 32) {
        out[lane] = mine;
        out[32 + lane] = digits;
    }
    return sum;
}

template <bool FULL, bool I32, int CH, int THREADS>
__global__ __launch_bounds__(THREADS) void k_planes(PlaneArgs a) {
    constexpr int WAVES = THREADS / 64;
    __shared__ uint32_t buf[16 * CH];
    __shared__ int32_t repeated;  // entries less columns set
    const int32_t count = FULL ? a.meta.ctr[0] : a.meta.ctr[1];
    if (!FULL && a.meta.ctr[2] != MODE_DENSE_U) return;
    const int32_t pitch = FULL ? a.pitch : a.meta.ctr[4];
    const int32_t chunks = (pitch + CH - 1) / CH;
    for (int64_t item = blockIdx.x; item < (int64_t)(count + 31) / 32 * chunks; item += gridDim.x) {
        const int64_t g = item / chunks;
        const int32_t c0 = (int32_t)(item % chunks) * CH;
        const int32_t cn = min(CH, pitch - c0);             // a multiple of 64
        const int32_t ncols = FULL ? a.m : a.meta.ctr[3];   // real columns: candidates or U
        const int32_t bits = FULL ? a.bits : rank_bits(a.meta.ctr[6]);
        const int32_t *srcs = FULL ? a.meta.full_src : a.meta.trunc_src;
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const int32_t live = (int32_t)min((int64_t)32, count - 32 * g);  // voters of this group

        for (int i = threadIdx.x; i < 16 * CH; i += THREADS) {
            const int p = i / CH;
            buf[i] = (2 * p < live ? 0xFFFFu : 0u) | (2 * p + 1 < live ? 0xFFFF0000u : 0u);
        }
        if (threadIdx.x == 0) repeated = 0;
        int32_t extra = 0;
        __syncthreads();
        uint16_t *half = reinterpret_cast<uint16_t *>(buf);
        for (int v = wave; v < live; v += WAVES) {  // a wavefront per ballot
            const int32_t src = srcs[32 * g + v];
            const int32_t k = a.meta.len[src];
            uint16_t *row = half + (v >> 1) * (2 * CH) + (v & 1);
            auto place = [&](int32_t t, int32_t id) {
                if ((uint32_t)id >= (uint32_t)a.m) return;  // reported by the scan
                const int32_t col = (FULL ? id : a.meta.umap[id]) - c0;
                if ((uint32_t)col >= (uint32_t)cn) return;
                row[2 * col] = (uint16_t)t;
                ++extra;
            };
            constexpr int FLY = 4;  // pieces per lane in flight
            const RowPieces<I32> pieces(a.ballots, a.n, a.L, src);
            const int32_t need = (pieces.head + k + pieces.PER - 1) / pieces.PER;
            for (int32_t j0 = 0; j0 < need; j0 += 64 * FLY) {
                v4u x[FLY];
                pieces.template load<FLY>(x, j0 + lane);
                for (int u = 0; u < FLY; ++u)
                    pieces.each(x[u], j0 + 64 * u + lane, k, [&](int32_t t, uint32_t raw) { place(t, (int32_t)raw); });
            }
        }
        __syncthreads();
        // the group's voters in the order of the planes' bits
        const uint32_t voters = voter_bits(live);
        extra += planes_out<CH, THREADS>(buf, cn, ncols - c0, voters, bits, pitch,
                                         a.planes + g * bits * (int64_t)pitch + c0);
        check_repeats(extra, &repeated, a.err);
        if (a.weight && c0 == 0 && wave == 0) {
            const int v = 2 * (lane & 15) + ((lane >> 4) & 1);  // the voter of bit `lane`
            const uint32_t sum = weight_planes(lane < 32 && v < live ? a.weight[srcs[32 * g + v]] : 0u,
                                               a.wplanes + WEIGHT_WORDS * g);
            if (FULL && lane == 0) atomicAdd(&a.meta.ctr[8], (int32_t)sum);
        }
        __syncthreads();  // the LDS is read
    }
}

// The planes of every ballot over all candidates, straight from the ballots
// (the one-pass count of small elections): the listed length is found on the
// way.  1024 threads and a group of 32 ballots, two ballots per wavefront
// with their first pieces loaded together.  (The code for weights is left out
// where there are none: with it the planes of n = 12124, m = 139 took 10.2 us,
// without 8.1.)
struct AllArgs {
    const void *ballots;
    int32_t n, L, m, pitch, bits;
    const uint32_t *weight;
    uint32_t *planes, *wplanes;
    int32_t *err;
    int32_t *repeated;  // where a repeated id is recorded: the error word, or a word that k_weight_total reports
};

template <bool I32, int CH, bool WEIGHTED>
__global__ __launch_bounds__(1024) void k_planes_all(AllArgs a) {
    using P = RowPieces<I32, true>;
    constexpr int FLY = 2;  // pieces per lane and ballot in flight
    __shared__ uint32_t buf[16 * CH];
    __shared__ int32_t repeated;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int32_t g = blockIdx.x, c0 = (int32_t)blockIdx.y * CH, cn = min(CH, a.pitch - c0);
    const int32_t live = min(32, a.n - 32 * g);
    v4u x[2][FLY];
#pragma unroll
    for (int h = 0; h < 2; ++h)
        P(a.ballots, a.n, a.L, 32 * g + min(wave + 16 * h, live - 1)).template load<FLY>(x[h], lane);
    for (int p = 0; p < 16; ++p) {
        const uint32_t fill = (2 * p < live ? 0xFFFFu : 0u) | (2 * p + 1 < live ? 0xFFFF0000u : 0u);
        for (int c = threadIdx.x; c < cn; c += 1024) buf[p * CH + c] = fill;
    }
    if (threadIdx.x == 0) repeated = 0;
    __syncthreads();
    int32_t extra = 0;
    bool bad = false;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int v = wave + 16 * h;
        if (v >= live) continue;
        const P row(a.ballots, a.n, a.L, 32 * g + v);
        int32_t k = a.L;  // first padding entry
        auto pads = [&](const v4u &p, int32_t j) {
            if (j < row.count && P::top(p) >= (uint32_t)a.m)
                row.each(p, j, a.L, [&](int32_t t, uint32_t raw) {
                    if (raw_id<I32>(raw) < 0) k = min(k, t);
                });
        };
        for (int u = 0; u < FLY; ++u) pads(x[h][u], 64 * u + lane);
        for (int32_t j = 64 * FLY + lane; j < row.count; j += 64) {
            v4u p[1];
            row.template load<1>(p, j);
            pads(p[0], j);
        }
        for (int off = 32; off >= 1; off >>= 1) k = min(k, __shfl_xor(k, off));
        uint16_t *out = reinterpret_cast<uint16_t *>(buf) + (v >> 1) * (2 * CH) + (v & 1);
        auto place = [&](int32_t t, uint32_t raw) {
            if (raw >= (uint32_t)a.m) {
                bad = true;
                return;
            }
            const int32_t c = (int32_t)raw - c0;
            if ((uint32_t)c >= (uint32_t)cn) return;
            out[2 * c] = (uint16_t)t;
            ++extra;
        };
        for (int u = 0; u < FLY; ++u) row.each(x[h][u], 64 * u + lane, k, place);
        for (int32_t j = 64 * FLY + lane; j < row.count; j += 64) {
            v4u p[1];
            row.template load<1>(p, j);
            row.each(p[0], j, k, place);
        }
    }
    if (bad) set_device_error(a.err, SCHULZE_EBALLOT);
    __syncthreads();
    extra += planes_out<CH, 1024>(buf, cn, a.m - c0, voter_bits(live), a.bits, a.pitch,
                                  a.planes + (int64_t)g * a.bits * a.pitch + c0);
    check_repeats(extra, &repeated, a.repeated);
    if (WEIGHTED && blockIdx.y == 0 && wave == 0) {
        const int v = 2 * (lane & 15) + ((lane >> 4) & 1);
        (void)weight_planes(lane < 32 && v < live ? a.weight[32 * g + v] : 0u, a.wplanes + WEIGHT_WORDS * g);
    }
}

// The same for short rows (L <= 64): 256 threads take a group's entries as
// one run, so that no lane idles on a ballot shorter than a wavefront (n =
// 180227 top-10 of m = 159: a wavefront per ballot took 100 us, this 16).
template <bool I32, int CH, bool WEIGHTED>
__global__ __launch_bounds__(256) void k_planes_short(AllArgs a) {
    constexpr int FLY = 8;  // entries per thread: 32 ballots of at most 64
    __shared__ uint32_t buf[16 * CH];
    __shared__ int32_t first[32];
    __shared__ int32_t repeated;
    const int32_t g = blockIdx.x, c0 = (int32_t)blockIdx.y * CH, cn = min(CH, a.pitch - c0);
    const int32_t live = min(32, a.n - 32 * g), entries = live * a.L;
    const int64_t base = (int64_t)32 * g * a.L;
    uint32_t x[FLY];
    for (int u = 0; u < FLY; ++u)  // (clamped: all in flight together)
        x[u] = load_raw<I32>(a.ballots, base + min((int32_t)threadIdx.x + 256 * u, entries - 1));
    for (int p = 0; p < 16; ++p) {
        const uint32_t fill = (2 * p < live ? 0xFFFFu : 0u) | (2 * p + 1 < live ? 0xFFFF0000u : 0u);
        for (int c = threadIdx.x; c < cn; c += 256) buf[p * CH + c] = fill;
    }
    if (threadIdx.x < 32) first[threadIdx.x] = a.L;
    if (threadIdx.x == 0) repeated = 0;
    __syncthreads();
    const uint32_t inv = (uint32_t)((0x100000000ull + (uint64_t)a.L - 1) / (uint64_t)a.L);  // entry / L for L > 1
    auto place_of = [&](int u, int32_t &v, int32_t &t) {
        const int32_t f = (int32_t)threadIdx.x + 256 * u;
        v = a.L > 1 ? (int32_t)__umulhi((uint32_t)f, inv) : f;
        t = f - v * a.L;
        return f < entries;
    };
    for (int u = 0; u < FLY; ++u) {
        int32_t v, t;
        if (place_of(u, v, t) && raw_id<I32>(x[u]) < 0) atomicMin(&first[v], t);
    }
    __syncthreads();
    int32_t extra = 0;
    bool bad = false;
    uint16_t *half = reinterpret_cast<uint16_t *>(buf);
    for (int u = 0; u < FLY; ++u) {
        int32_t v, t;
        if (!place_of(u, v, t) || t >= first[v]) continue;
        if (x[u] >= (uint32_t)a.m) {
            bad = true;
            continue;
        }
        const int32_t c = (int32_t)x[u] - c0;
        if ((uint32_t)c >= (uint32_t)cn) continue;
        half[(v >> 1) * (2 * CH) + 2 * c + (v & 1)] = (uint16_t)t;
        ++extra;
    }
    if (bad) set_device_error(a.err, SCHULZE_EBALLOT);
    __syncthreads();
    extra += planes_out<CH, 256>(buf, cn, a.m - c0, voter_bits(live), a.bits, a.pitch,
                                 a.planes + (int64_t)g * a.bits * a.pitch + c0);
    check_repeats(extra, &repeated, a.repeated);
    if (WEIGHTED && blockIdx.y == 0 && threadIdx.x < 64) {
        const int lane = threadIdx.x, v = 2 * (lane & 15) + ((lane >> 4) & 1);
        (void)weight_planes(lane < 32 && v < live ? a.weight[32 * g + v] : 0u, a.wplanes + WEIGHT_WORDS * g);
    }
}

template <bool I32, bool WEIGHTED>
int planes_all(schulze_ctx *ctx, hipStream_t s, const AllArgs &pa, int64_t groups) {
    const int ch = pa.L <= 64 ? (pa.pitch <= 128 ? 128 : 512) : (pa.pitch <= 512 ? 512 : 2048);
    const dim3 pg((unsigned)groups, (unsigned)ceil_div(pa.pitch, ch));
    if (ch == 128)
        SCHULZE_LAUNCH(ctx, K_BALLOT_SCATTER, s, (k_planes_short<I32, 128, WEIGHTED><<<pg, dim3(256), 0, s>>>(pa)));
    else if (pa.L <= 64)
        SCHULZE_LAUNCH(ctx, K_BALLOT_SCATTER, s, (k_planes_short<I32, 512, WEIGHTED><<<pg, dim3(256), 0, s>>>(pa)));
    else if (ch == 512)
        SCHULZE_LAUNCH(ctx, K_BALLOT_SCATTER, s, (k_planes_all<I32, 512, WEIGHTED><<<pg, dim3(1024), 0, s>>>(pa)));
    else
        SCHULZE_LAUNCH(ctx, K_BALLOT_SCATTER, s, (k_planes_all<I32, 2048, WEIGHTED><<<pg, dim3(1024), 0, s>>>(pa)));
    return SCHULZE_OK;
}

// ------------------------------------------------------------------ bit-plane count
// Persistent kernel.  Work units are (tile of CT x CT candidates, group of
// 32 voters); each workgroup takes a contiguous range of units (equal work
// per workgroup).  A tile whose groups are all counted by one workgroup goes
// straight into acc; the others' counts (at most the first and the last tile
// of a range) go to that workgroup's two slots of partial tiles, which
// k_count_reduce adds up: 64 KB written per slot, where device-wide atomics
// into acc took 0.5 us per flushed tile for the whole chip (m = 1023,
// n = 12007: 431 us, of which the counting is about 90).
//   COUNT_FULL  full rankings, tiles X <= Y over candidates; acc also takes
//               d[y][x] = voters - d[x][y].
//   COUNT_U     truncated ballots over U space, all tiles (X, Y); U indices
//               map back through ulist; the sentinel column y = |U| gives
//               R[x].
//   COUNT_ALL   every ballot over all candidates, all tiles; the counts are
//               final and go to d (small elections: see count_all).
// Bound by the vector ALU: a thread carries 8 x 8 masks and counts, so a
// bit takes 64 v_bitop3_b32 and four 16-byte LDS reads (8 row and 8 column
// words), and the reads' 32 cycles per wavefront and bit hide behind the
// products of the other wavefronts (three per SIMD).  At m = 4096, n = 42000:
// 90 T comparisons/s (the packed subtractions: 31 T); larger thread tiles
// (16 x 8, counts packed in 16 bits) had fewer reads per mask but two
// wavefronts per SIMD: 10% slower.
enum CountMode { COUNT_FULL, COUNT_U, COUNT_ALL };

struct DenseArgs {
    const uint32_t *planes;
    int32_t pitch, bits;  // full rankings (pitch a multiple of CT)
    int32_t m;
    Meta meta;
    uint32_t *acc;  // m x m
    int64_t lda;
    uint32_t *rsum;
    const uint32_t *wplanes;  // with voter weights
    uint32_t *partial;        // two CT x CT tiles per workgroup (COUNT_ALL: one per workgroup and tile)
    // COUNT_ALL
    int32_t n;
    int32_t whole;  // every workgroup counts whole tiles
    void *d;
    int64_t ldd;
    int32_t d32;
    uint32_t limit;
    int32_t *err;
};

// The units of a count and their division among the workgroups.
struct CountPlan {
    int32_t nvoters, groups, pitch, nb, nu;
    int32_t whole;
    int64_t ntiles, units, workers;
    __device__ int64_t first(int64_t w) const {
        return whole ? ntiles * w / workers * groups : units * w / workers;
    }
};
template <int MODE>
__device__ inline CountPlan count_plan(const DenseArgs &a, int32_t grid) {
    CountPlan c;
    c.nvoters = MODE == COUNT_ALL ? a.n : MODE == COUNT_U ? a.meta.ctr[1] : a.meta.ctr[0];
    c.groups = (c.nvoters + 31) / 32;  // units per tile
    c.pitch = MODE == COUNT_U ? a.meta.ctr[4] : a.pitch;
    c.nu = MODE == COUNT_U ? a.meta.ctr[3] : a.m;
    c.nb = c.pitch / CT;
    c.ntiles = MODE == COUNT_FULL ? (int64_t)c.nb * (c.nb + 1) / 2 : (int64_t)c.nb * c.nb;
    // ranges of at least four units (writing and adding up a partial tile
    // costs about as much as one); COUNT_ALL is launched with its workers
    c.units = c.ntiles * c.groups;
    c.whole = MODE == COUNT_ALL && a.whole;
    c.workers = MODE == COUNT_ALL ? grid : min((int64_t)grid, (c.units + 3) / 4);
    return c;
}

// Voters (their weight) that a full-ranking tile's mirror takes d[y][x] from.
template <bool WEIGHTED>
__device__ inline uint32_t full_total(const DenseArgs &a) {
    return (uint32_t)(WEIGHTED ? a.meta.ctr[8] : a.meta.ctr[0]);
}

// cnt voters prefer x to y (indices of the count): into acc, and for full
// rankings outside diagonal tiles the mirror too.  One thread per element
// and launch: plain additions.
template <int MODE>
__device__ inline void add_count(const DenseArgs &a, int32_t nu, int32_t x, int32_t y, bool mirror, uint32_t total,
                                 uint32_t cnt, bool &over) {
    if (MODE == COUNT_U) {
        if (x >= nu || y > nu) return;
        const int32_t gx = a.meta.ulist[x];
        if (y == nu)
            a.rsum[gx] += cnt;
        else if (x != y)
            a.acc[(int64_t)gx * a.lda + a.meta.ulist[y]] += cnt;
    } else if (x >= nu || y >= nu) {
        return;
    } else if (MODE == COUNT_ALL) {  // (ranks equal to themselves: the diagonal is 0)
        over |= cnt > a.limit;
        const uint32_t v = min(cnt, a.limit);
        if (a.d32)
            static_cast<uint32_t *>(a.d)[(int64_t)x * a.ldd + y] = v;
        else
            static_cast<uint16_t *>(a.d)[(int64_t)x * a.ldd + y] = (uint16_t)v;
    } else if (x != y) {
        a.acc[(int64_t)x * a.lda + y] += cnt;
        if (mirror) a.acc[(int64_t)y * a.lda + x] += total - cnt;
    }
}

__device__ inline void tri_coords(int32_t t, int32_t nb, int32_t &X, int32_t &Y) {
    int32_t x = 0, start = 0;
    while (start + (nb - x) <= t) {
        start += nb - x;
        ++x;
    }
    X = x;
    Y = x + (t - start);
}

// acc += the masks' voters' weights times 2^shift, sixteen bits of them as the
// digits of four bits in d: a mask is spread to one bit per digit (seven
// operations), then four v_dot8_u32_u4 per digit and a shifted addition, 27
// operations where bit planes take 48.
__device__ __forceinline__ void add_digits(const Masks &lt, const uint32_t (&d)[16], int shift, uint32_t (&acc)[8][8]) {
    uint32_t k = 0x11111111u, one = 1u, two = 2u, three = 3u;
    asm volatile("" : "+s"(k), "+s"(one), "+s"(two), "+s"(three));  // (spread masks are not kept for the next call)
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t m = lt.get(i, j);
            const uint32_t x[4] = {m & k, (m >> one) & k, (m >> two) & k, (m >> three) & k};
            uint32_t sum = 0u;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                uint32_t t = 0u;
#pragma unroll
                for (int q = 0; q < 4; ++q) t = __builtin_amdgcn_udot8(x[q], d[4 * p + q], t, false);
                sum += t << (4 * p);
            }
            acc[i][j] += sum << shift;
            __builtin_amdgcn_sched_barrier(0);  // one mask at a time: few registers
        }
}

// Bits of the weights that are added up as digits, sixteen at a time; the bits
// above go plane by plane.  (Of sixteen bits or what is left, planes are fewer
// operations up to 8.)
__host__ __device__ inline int32_t digit_bits(int32_t bits) { return bits % 16 > 8 ? bits / 16 * 16 + 16 : bits / 16 * 16; }
// Operations per mask for weights of so many bits.
inline int32_t weight_ops(int32_t bits) {
    const int32_t digits = digit_bits(bits);
    return 27 * (digits / 16) + 3 * std::max(bits - digits, 0);
}

template <int MODE, bool WEIGHTED>
__global__ __launch_bounds__(256, 3) void k_count_bits(DenseArgs a) {
    constexpr int ROW = 2 * CT;  // LDS words per bit: the tile's rows, then its columns
    __shared__ __attribute__((aligned(16))) uint32_t lds[2 * MAX_BITS * ROW];
    if (MODE == COUNT_U && a.meta.ctr[2] != MODE_DENSE_U) return;
    CNT_LDS uint32_t *st = (CNT_LDS uint32_t *)lds;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the thread index, opaque: what the staging and the flush build from it
    // is computed there, not kept in registers through the counting
    auto thread = [] {
        int i = (int)threadIdx.x;
        asm volatile("" : "+v"(i));
        return i;
    };
    const CountPlan c = count_plan<MODE>(a, gridDim.x);
    if (blockIdx.x >= c.workers) return;
    const int32_t groups = c.groups, pitch = c.pitch, nb = c.nb;
    const int32_t bits = MODE == COUNT_U ? rank_bits(a.meta.ctr[6]) : a.bits;
    const int32_t wbits = WEIGHTED && a.meta.ctr[7] ? 32 - __clz(a.meta.ctr[7]) : 0;
    const int64_t u0 = c.first(blockIdx.x), u1 = c.first(blockIdx.x + 1);

    // a thread counts rows ty * 4 + (0 .. 3) and 64 + ty * 4 + (0 .. 3) of
    // the tile, and columns likewise by tx: its 16-byte LDS reads are then
    // contiguous over the lanes
    uint32_t acc[8][8];
    for (int i = 0; i < 8; ++i)
        for (int j = 0; j < 8; ++j) acc[i][j] = 0u;
    const int32_t t0 = (int32_t)(u0 / groups);
    int32_t t = t0, X, Y;
    int32_t g = (int32_t)(u0 % groups), seg0 = g;
    auto coords = [&](int32_t tile, int32_t &tX, int32_t &tY) {
        if (MODE != COUNT_FULL) {
            tX = tile / nb;
            tY = tile % nb;
        } else {
            tri_coords(tile, nb, tX, tY);
        }
    };
    // group sg of tile (tX, tY) to buffer sb: one wavefront instruction per
    // bit, lanes 0 .. 31 the tile's rows, 32 .. 63 its columns
    auto stage = [&](int32_t tX, int32_t tY, int32_t sg, int sb) {
        const uint32_t *src = a.planes + (int64_t)sg * bits * pitch;
        const int lane = thread() & 63;
        const uint32_t off = lane < 32 ? tX * CT + 4 * lane : tY * CT + 4 * (lane - 32);
        for (int b = wave; b < bits; b += 4)
            __builtin_amdgcn_global_load_lds(src + (int64_t)b * pitch + off, st + (sb * MAX_BITS + b) * ROW, 16, 0, 0);
    };
    auto flush = [&](int32_t seg1) {
        const int ftx = thread() & 15, fty = thread() >> 4;
        if (MODE == COUNT_ALL ? c.whole : seg0 == 0 && seg1 == groups) {
            const uint32_t total = MODE == COUNT_FULL ? full_total<WEIGHTED>(a) : 0u;
            bool over = false;
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    add_count<MODE>(a, c.nu, X * CT + (i & 4) * 16 + fty * 4 + (i & 3),
                                    Y * CT + (j & 4) * 16 + ftx * 4 + (j & 3), X != Y, total, acc[i][j], over);
            if (MODE == COUNT_ALL && over) set_device_error(a.err, SCHULZE_ERANGE);
        } else {
            const int64_t slot = MODE == COUNT_ALL ? (int64_t)blockIdx.x + t : (int64_t)blockIdx.x * 2 + (t != t0);
            uint32_t *out = a.partial + slot * (CT * CT);
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int j = 0; j < 8; j += 4)
                    *reinterpret_cast<uint4 *>(out + ((i & 4) * 16 + fty * 4 + (i & 3)) * CT + (j & 4) * 16 + ftx * 4) =
                        make_uint4(acc[i][j], acc[i][j + 1], acc[i][j + 2], acc[i][j + 3]);
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[i][j] = 0u;
    };

    coords(t, X, Y);
    stage(X, Y, g, 0);
    for (int64_t u = u0; u < u1; ++u) {
        const int sb = (int)((u - u0) & 1);
        __builtin_amdgcn_s_waitcnt(0);  // this wavefront's pieces of unit u are in LDS
        __syncthreads();                // everyone's are, and unit u-1 is consumed
        int32_t nX = X, nY = Y;
        int32_t ng = g + 1;
        if (ng == groups) {
            ng = 0;
            if (u + 1 < u1) coords(t + 1, nX, nY);
        }
        if (u + 1 < u1) stage(nX, nY, ng, sb ^ 1);

        const CNT_LDS uint32_t *rows = st + sb * MAX_BITS * ROW;
        Masks lt;
        lt.clear();
        struct Bit {
            v4u x[2], y[2];
        };
        auto read = [&](int b, Bit &q) {
            const CNT_LDS uint32_t *r = rows + b * ROW;
            q.x[0] = *(const CNT_LDS v4u *)(r + ty * 4);
            q.x[1] = *(const CNT_LDS v4u *)(r + 64 + ty * 4);
            q.y[0] = *(const CNT_LDS v4u *)(r + CT + tx * 4);
            q.y[1] = *(const CNT_LDS v4u *)(r + CT + 64 + tx * 4);
        };
        // the next bit's reads are issued before the products of this one
        // (the scheduling barriers keep them there)
        Bit q0, q1;
        read(0, q0);
#pragma unroll 1
        for (int b = 0; b + 1 < bits; b += 2) {
            read(b + 1, q1);
            __builtin_amdgcn_sched_barrier(0);
            lt.step(q0.x, q0.y);
            __builtin_amdgcn_sched_barrier(0);
            read(b + 2 < bits ? b + 2 : 0, q0);
            __builtin_amdgcn_sched_barrier(0);
            lt.step(q1.x, q1.y);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (bits & 1) lt.step(q0.x, q0.y);
        if constexpr (WEIGHTED) {
            const uint32_t *wp = a.wplanes + (int64_t)WEIGHT_WORDS * g;
            const int32_t digits = digit_bits(wbits);
#pragma unroll 1
            for (int32_t b = 0; b < digits; b += 16) {
                uint32_t d[16], any = 0u;
#pragma unroll
                for (int q = 0; q < 16; ++q) any |= d[q] = __builtin_amdgcn_readfirstlane(wp[32 + b + q]);
                if (any == 0u) continue;
                add_digits(lt, d, b, acc);
            }
#pragma unroll 1
            for (int32_t b = digits; b < wbits; ++b) {
                const uint32_t wm = __builtin_amdgcn_readfirstlane(wp[b]);
                if (wm == 0u) continue;
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[i][j] += (uint32_t)__popc(lt.get(i, j) & wm) << b;
            }
        } else {
            lt.count(acc);
        }
        if (ng == 0 || u + 1 == u1) {
            flush(g + 1);
            seg0 = 0;
            if (ng == 0) ++t;
        }
        X = nX;
        Y = nY;
        g = ng;
    }
}

// The partial tiles of tile t, those of the workgroups w0 .. w1 whose ranges
// meet it, the first in slot s0 (a workgroup's slot: twice its number for its
// first tile, the next one for its last; in COUNT_ALL its number plus t).
struct TileParts {
    int64_t w0, w1, s0;
};
template <int MODE>
__device__ inline TileParts tile_parts(const CountPlan &c, int32_t t) {
    const int64_t ub = (int64_t)t * c.groups, ue = ub + c.groups;
    TileParts q{ub * c.workers / c.units, (ue - 1) * c.workers / c.units, 0};
    while (c.first(q.w0 + 1) <= ub) ++q.w0;
    while (c.first(q.w0) > ub) --q.w0;
    while (c.first(q.w1 + 1) < ue) ++q.w1;
    while (c.first(q.w1) >= ue) --q.w1;
    q.s0 = MODE == COUNT_ALL ? q.w0 + t : 2 * q.w0 + (c.first(q.w0) < ub);
    return q;
}

// The partial tiles added up.  With few per tile, a workgroup takes 32 rows
// of a tile and the mirror of a full-ranking tile goes through LDS, so that
// both are written along rows; with many (few tiles, many voters), two rows,
// and the four wavefronts share the partial tiles out (one thread adding 391
// of them took 400 us).
template <int MODE, bool WEIGHTED>
__global__ __launch_bounds__(256) void k_count_reduce(DenseArgs a, int32_t grid) {
    __shared__ uint32_t buf[32][CT + 1];
    if (MODE == COUNT_U && a.meta.ctr[2] != MODE_DENSE_U) return;
    const CountPlan c = count_plan<MODE>(a, grid);
    if (c.units == 0) return;
    const uint32_t total = MODE == COUNT_FULL ? full_total<WEIGHTED>(a) : 0u;
    constexpr int64_t STEP = MODE == COUNT_ALL ? 1 : 2;  // slots per workgroup
    bool over = false;
    const bool many = c.workers > 4 * c.ntiles;
    const int32_t rows = many ? 2 : 32, per = CT / rows;  // rows of a piece, pieces of a tile
    for (int64_t q = blockIdx.x; q < per * c.ntiles; q += gridDim.x) {
        const int32_t t = (int32_t)(q / per), r0 = (int32_t)(q % per) * rows;
        const TileParts parts = tile_parts<MODE>(c, t);
        if (MODE != COUNT_ALL && parts.w0 == parts.w1) continue;  // counted whole, in acc already
        int32_t X, Y;
        if (MODE != COUNT_FULL) {
            X = t / c.nb;
            Y = t % c.nb;
        } else {
            tri_coords(t, c.nb, X, Y);
        }
        const int64_t s1 = STEP * parts.w1 + (MODE == COUNT_ALL ? t : 0);
        // slots of the parts after the first: STEP apart up to s1
        const int64_t s2 = MODE == COUNT_ALL ? parts.s0 + 1 : 2 * parts.w0 + 2;
        __syncthreads();  // the last piece's LDS has been read
        if (many) {
            const int col = (threadIdx.x & 31) * 4, row = (threadIdx.x >> 5) & 1, wave = threadIdx.x >> 6;
            const uint32_t *p = a.partial + (r0 + row) * CT + col;
            uint32_t v[4] = {};
            auto add = [&](int64_t slot) {
                const uint4 x = *reinterpret_cast<const uint4 *>(p + slot * (CT * CT));
                v[0] += x.x, v[1] += x.y, v[2] += x.z, v[3] += x.w;
            };
            if (wave == 0) add(parts.s0);
#pragma unroll 8
            for (int64_t sl = s2 + STEP * wave; sl <= s1; sl += 4 * STEP) add(sl);
            for (int e = 0; e < 4; ++e) buf[wave * 2 + row][col + e] = v[e];
            __syncthreads();
            if (wave == 0)
                for (int e = 0; e < 4; ++e)
                    add_count<MODE>(a, c.nu, X * CT + r0 + row, Y * CT + col + e, X != Y, total,
                                    buf[row][col + e] + buf[2 + row][col + e] + buf[4 + row][col + e] +
                                        buf[6 + row][col + e],
                                    over);
            continue;
        }
        const int col = (threadIdx.x & 31) * 4, row = threadIdx.x >> 5;
        uint32_t v[4][4] = {};
        auto add = [&](int64_t slot) {
            const uint32_t *p = a.partial + slot * (CT * CT) + r0 * CT + col;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint4 x = *reinterpret_cast<const uint4 *>(p + (row + 8 * k) * CT);
                v[k][0] += x.x, v[k][1] += x.y, v[k][2] += x.z, v[k][3] += x.w;
            }
        };
        add(parts.s0);
#pragma unroll 2
        for (int64_t sl = s2; sl <= s1; sl += STEP) add(sl);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                add_count<MODE>(a, c.nu, X * CT + r0 + row + 8 * k, Y * CT + col + e, false, 0u, v[k][e], over);
                if (MODE == COUNT_FULL) buf[row + 8 * k][col + e] = v[k][e];
            }
        if (MODE != COUNT_FULL || X == Y) continue;
        __syncthreads();
        for (int i = threadIdx.x; i < 32 * CT; i += 256) {
            const int32_t x = X * CT + r0 + (i & 31), y = Y * CT + (i >> 5);
            if (x < c.nu && y < c.nu) a.acc[(int64_t)y * a.lda + x] += total - buf[i & 31][i >> 5];
        }
    }
    if (MODE == COUNT_ALL && over) set_device_error(a.err, SCHULZE_ERANGE);
}

// ------------------------------------------------------------------ pair scattering
// One wavefront per truncated ballot: lane t handles listed entry t.  For
// every earlier entry i < t the pair (c_i before c_t) adds the voter's
// weight to C[c_i][c_t], i.e. subtracts it from acc[c_t][c_i]; every listed
// entry adds the weight to R.  Equal entries are a repeated id.
template <bool I32>
__global__ __launch_bounds__(256) void k_count_pairs(const void *__restrict__ ballots, int32_t L,
                                                     int32_t m, const uint32_t *__restrict__ weight, Meta meta,
                                                     uint32_t *__restrict__ acc, int64_t lda,
                                                     uint32_t *__restrict__ rsum, int32_t *err) {
    if (meta.ctr[2] != MODE_SPARSE) return;
    const int lane = threadIdx.x & 63;
    const int64_t slot = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (slot >= meta.ctr[1]) return;
    const int32_t v = meta.trunc_src[slot];
    const int32_t k = meta.len[v];
    const uint32_t w = weight ? weight[v] : 1u;
    const int64_t base = (int64_t)v * L;
    bool dup = false;
    for (int t = lane; t < k; t += 64) {
        const int32_t ct = read_id<I32>(ballots, base + t);
        if (ct < 0 || ct >= m) continue;  // reported by the scan
        if (w) atomicAdd(&rsum[ct], w);
        uint32_t *row = acc + (int64_t)ct * lda;
        for (int i = 0; i < t; ++i) {
            const int32_t ci = read_id<I32>(ballots, base + i);
            if (ci == ct) dup = true;
            if (w && ci >= 0 && ci < m) atomicSub(&row[ci], w);
        }
    }
    if (__ballot(dup) && lane == 0) set_device_error(err, SCHULZE_EBALLOT);
}

// ------------------------------------------------------------------ bucketed pair counting
// The same sums as k_count_pairs without its random device-wide atomics into
// the m x m accumulator.  The listed entries ("occurrences") of truncated
// ballots are bucketed by candidate (a counting sort: per-workgroup
// histograms in LDS over fixed ballot ranges, column prefixes, placement),
// and then each candidate r's row of C^T (C[y][r] = weight of ballots
// listing y before r) is accumulated in LDS from the ballot prefixes ahead
// of its occurrences; d[r][y] = R_r - C[y][r] (plus any full-ranking
// counts).  A candidate with at most its chunk of occurrences is one work item
// that writes its row of d at once; a heavier one is split into items that
// write their partial rows to a buffer, summed by the finish.  Nothing here
// needs the m x m accumulator unless full rankings are counted as well.
// Occurrences per accumulation item (at most 65535: packed counts): a quarter
// of a workgroup's share of all, so that one item does not outlast the rest,
// within these bounds (a heavier candidate's items each write a partial row).
constexpr int OCC_CHUNK_MIN = 1024, OCC_CHUNK_MAX = 8192;
constexpr int32_t OCC_MAX_M = 32768;       // an LDS row of counts
constexpr int64_t OCC_MAX = (int64_t)1 << 27;  // occurrence buffer limit (entries)
constexpr int OCC_FIN_COLS = 2048;         // columns per unit of the finish
constexpr int OCC_QUEUES = 8, TICKET_STRIDE = 64;
constexpr uint32_t NO_PARTIAL = 0xFFFFFFFFu;  // the only item of its row
constexpr int FIN_COUNT = 5;               // meta.ctr slot: rows listed for the finish

struct OccArgs {
    const void *ballots;
    int dtype32;
    int32_t L, m;
    int64_t n;
    int32_t tbits;        // occurrence word: ballot << tbits | position
    const uint32_t *weight;
    Meta meta;
    uint32_t *hist;       // G x m: per-workgroup counts, then their exclusive prefix over workgroups
    uint32_t *row_start;  // m + 1: occurrences per candidate, then the exclusive scan
    uint4 *items;         // accumulation items: candidate, its occurrences [begin, end), partial row or NO_PARTIAL
    uint32_t *item_start; // m + 1: accumulation items, exclusive scan
    uint32_t *tickets;    // OCC_QUEUES counters of items handed out, TICKET_STRIDE words apart
    uint32_t chunk;       // occurrences per accumulation item
    uint32_t *part_start; // m + 1: partial rows per candidate (its items if more than one), then the scan
    int32_t *fin;         // candidates whose rows the finish writes (no occurrences, or two or more items);
                          // their number in meta.ctr[FIN_COUNT]
    uint32_t *occ;        // placed occurrences
    void *partial;        // partial rows, pitch ppitch elements (uint16 for unit weights, else uint32)
    int64_t ppitch;
    uint32_t *acc;
    int64_t lda;
    uint32_t *rsum;
    int32_t *err;
};

// Eight consecutive values of a row of d: 16-byte stores (at any alignment)
// when all eight columns exist, else one at a time.
template <typename T>
__device__ inline void store8(T *__restrict__ drow, int32_t y, int32_t m, const uint32_t (&v)[8]) {
    if (y + 8 <= m) {
        if constexpr (sizeof(T) == 4) {
            tio::store16<T>(drow + y, make_uint4(v[0], v[1], v[2], v[3]));
            tio::store16<T>(drow + y + 4, make_uint4(v[4], v[5], v[6], v[7]));
        } else {
            tio::store16<T>(drow + y, make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16),
                                                 v[6] | (v[7] << 16)));
        }
        return;
    }
    for (int u = 0; u < 8 && y + u < m; ++u) drow[y + u] = (T)v[u];
}

// Ballots of bucketing workgroup g: [v0, v1) (the same in both passes).
__device__ inline void occ_range(int64_t n, int64_t &v0, int64_t &v1) {
    v0 = n * blockIdx.x / gridDim.x;
    v1 = n * (blockIdx.x + 1) / gridDim.x;
}

// PLACE = false: hist[g][c] = occurrences of c in workgroup g's ballots.
// PLACE = true:  write them to occ[] at row_start[c] + hist[g][c] + k.
// Rows of L <= 64 entries: a wavefront takes 64 / L ballots at once, one
// lane per entry; a ballot ends at its first padding entry (a wavefront
// ballot of the padding lanes gives it), and full rankings (m - 1 or more
// listed) are left to the dense count.  Longer rows: one ballot per
// wavefront, 64 entries at a time.
template <int MAXM, bool PLACE, bool I32>
__global__ __launch_bounds__(256) void k_occ_bucket(OccArgs a) {
    __shared__ uint32_t cnt[MAXM];
    if (a.meta.ctr[2] != MODE_SPARSE) return;
    const int32_t m = a.m, L = a.L;
    const int64_t hrow = (int64_t)blockIdx.x * m;
    if (PLACE) {
        // the workgroup's first slot per candidate, PRO candidates per thread
        // with every load in flight at once (one at a time, the loads took
        // most of the pass)
        constexpr int PRO = 16;
        for (int32_t c0 = threadIdx.x; c0 < m; c0 += 256 * PRO) {
            uint32_t rs[PRO], hs[PRO];
            for (int u = 0; u < PRO; ++u) {
                const int32_t c = c0 + 256 * u < m ? c0 + 256 * u : 0;
                rs[u] = a.row_start[c];
                hs[u] = a.hist[hrow + c];
            }
            for (int u = 0; u < PRO; ++u)
                if (c0 + 256 * u < m) cnt[c0 + 256 * u] = rs[u] + hs[u];
        }
    } else {
        for (int32_t c = threadIdx.x; c < m; c += 256) cnt[c] = 0u;
    }
    __syncthreads();
    int64_t v0, v1;
    occ_range(a.n, v0, v1);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto put = [&](int64_t v, int32_t t, int32_t c) {
        const uint32_t q = atomicAdd(&cnt[c], 1u);
        if (PLACE) a.occ[q] = ((uint32_t)v << a.tbits) | (uint32_t)t;
    };
    if (L <= 64) {
        const int32_t bpw = 64 / L;  // ballots per wavefront step
        const int32_t sub = lane / L, t = lane - sub * L;
        const bool lane_ok = sub < bpw;
        const uint64_t lane_bits = (L == 64) ? ~0ull : ((1ull << L) - 1ull);
        constexpr int U = 4;  // steps in flight
        for (int64_t vb = v0 + (int64_t)wave * bpw; vb < v1; vb += (int64_t)4 * bpw * U) {
            int32_t c[U];
            int64_t vv[U];
            for (int u = 0; u < U; ++u) {
                vv[u] = vb + (int64_t)4 * bpw * u + sub;
                // (every lane loads: a load under a condition is waited for inside it)
                c[u] = (int32_t)load_raw<I32>(a.ballots, lane_ok && vv[u] < v1 ? vv[u] * L + t : 0);
            }
            for (int u = 0; u < U; ++u) c[u] = lane_ok && vv[u] < v1 ? raw_id<I32>((uint32_t)c[u]) : -2;
            for (int u = 0; u < U; ++u) {
                const uint64_t pad = __ballot(c[u] < 0);  // -1 padding, -2 no ballot
                const uint64_t mine = lane_ok ? (pad >> (sub * L)) & lane_bits : lane_bits;
                const int32_t k = mine ? (int32_t)__builtin_ctzll(mine) : L;
                if (c[u] >= 0 && c[u] < m && t < k && k < m - 1) put(vv[u], t, c[u]);
            }
        }
    } else {
        for (int64_t v = v0 + wave; v < v1; v += 4) {
            const int32_t k = a.meta.len[v];
            if (k >= m - 1) continue;
            for (int32_t t = lane; t < k; t += 64) {
                const int32_t c = read_id<I32>(a.ballots, v * L + t);
                if (c >= 0 && c < m) put(v, t, c);
            }
        }
    }
    if (!PLACE) {
        __syncthreads();
        for (int32_t c = threadIdx.x; c < m; c += 256) a.hist[hrow + c] = cnt[c];
    } else {
        // the accumulation items, a candidate per thread
        for (int32_t c = blockIdx.x * 256 + threadIdx.x; c < m; c += gridDim.x * 256) {
            const uint32_t begin = a.row_start[c], end = a.row_start[c + 1], i0 = a.item_start[c];
            const uint32_t n = a.item_start[c + 1] - i0, p0 = a.part_start[c];
            for (uint32_t i = 0; i < n; ++i) {
                const uint32_t b = begin + i * a.chunk;
                a.items[i0 + i] = make_uint4((uint32_t)c, b, min(end, b + a.chunk), n > 1 ? p0 + i : NO_PARTIAL);
            }
        }
    }
}

// 64 candidates per workgroup, the G histogram rows split over COL_GROUPS
// thread groups (enough loads in flight to stream the histograms):
// hist[g][c] becomes its exclusive prefix over g; per candidate c,
// row_start[c] = occurrences, and the candidates whose rows the finish writes
// are listed.
constexpr int COL_GROUPS = 16;
__global__ __launch_bounds__(64 * COL_GROUPS) void k_occ_columns(OccArgs a, int32_t G) {
    __shared__ uint32_t part[COL_GROUPS][64];
    if (a.meta.ctr[2] != MODE_SPARSE) return;
    const int32_t c = blockIdx.x * 64 + (threadIdx.x & 63);
    const int grp = threadIdx.x >> 6;
    const int32_t g0 = G * grp / COL_GROUPS, g1 = G * (grp + 1) / COL_GROUPS;
    uint32_t sum = 0;
    if (c < a.m)
        for (int32_t g = g0; g < g1; ++g) sum += a.hist[(int64_t)g * a.m + c];
    part[grp][threadIdx.x & 63] = sum;
    __syncthreads();
    if (c >= a.m) return;
    uint32_t run = 0;
    for (int q = 0; q < grp; ++q) run += part[q][threadIdx.x & 63];
    for (int32_t g = g0; g < g1; ++g) {
        const uint32_t h = a.hist[(int64_t)g * a.m + c];
        a.hist[(int64_t)g * a.m + c] = run;
        run += h;
    }
    if (grp == COL_GROUPS - 1) {
        const uint32_t items = (run + a.chunk - 1) / a.chunk;
        a.row_start[c] = run;
        if (items != 1) a.fin[atomicAdd(&a.meta.ctr[FIN_COUNT], 1)] = c;
    }
}

// One workgroup of 1024 threads: from the occurrences per candidate in
// row_start, the exclusive prefixes of occurrences, accumulation items and
// partial rows, totals at [m].  A thread takes `per` consecutive candidates
// (a multiple of 4, at most 4 SCAN_VEC) as 16-byte loads that are all in
// flight together; the three sums go through wavefront shuffles and one LDS
// step (m = 32768: 30 us; three arrays read, three LDS scans of ten
// barriers each: 78 us).
constexpr int SCAN_VEC = 8;
static_assert(4 * SCAN_VEC * 1024 >= OCC_MAX_M, "candidates per thread of the scan");
__global__ __launch_bounds__(1024) void k_occ_scan(OccArgs a) {
    __shared__ uint32_t part[3][16];
    if (a.meta.ctr[2] != MODE_SPARSE) return;
    const int32_t m = a.m;
    const int32_t groups = (m + 4095) / 4096;  // of four candidates per thread
    const int32_t c0 = 4 * groups * (int32_t)threadIdx.x;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint4 v[SCAN_VEC];  // (the array's rows are padded to 256 bytes)
#pragma unroll
    for (int k = 0; k < SCAN_VEC; ++k) {
        const int32_t c = c0 + 4 * k;
        v[k] = reinterpret_cast<const uint4 *>(a.row_start)[k < groups && c < m ? c / 4 : 0];
    }
    uint32_t s[3] = {0u, 0u, 0u};
    const uint32_t chunk = a.chunk;
    auto items_of = [chunk](uint32_t occ) { return (occ + chunk - 1) / chunk; };
    auto count = [&](uint32_t occ) {
        const uint32_t it = items_of(occ);
        s[0] += occ;
        s[1] += it;
        s[2] += it > 1 ? it : 0u;
    };
#pragma unroll
    for (int k = 0; k < SCAN_VEC; ++k) {
        const int32_t c = c0 + 4 * k;
        if (k >= groups || c >= m) v[k] = make_uint4(0u, 0u, 0u, 0u);
        if (c + 1 >= m) v[k].y = 0u;
        if (c + 2 >= m) v[k].z = 0u;
        if (c + 3 >= m) v[k].w = 0u;
        count(v[k].x), count(v[k].y), count(v[k].z), count(v[k].w);
    }
    uint32_t run[3];  // inclusive over the wavefront, then exclusive over all
    for (int q = 0; q < 3; ++q) {
        run[q] = s[q];
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t o = __shfl_up(run[q], off);
            run[q] += lane >= off ? o : 0u;
        }
        if (lane == 63) part[q][wv] = run[q];
    }
    __syncthreads();
    for (int q = 0; q < 3; ++q) {
        run[q] -= s[q];
        for (int w = 0; w < wv; ++w) run[q] += part[q][w];
    }
    uint32_t *const dst[3] = {a.row_start, a.item_start, a.part_start};
#pragma unroll
    for (int k = 0; k < SCAN_VEC; ++k) {
        const int32_t c = c0 + 4 * k;
        if (k >= groups || c >= m) break;
        const uint32_t x[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
        uint32_t o[3][4];
        for (int u = 0; u < 4; ++u) {
            for (int q = 0; q < 3; ++q) o[q][u] = run[q];
            const uint32_t it = items_of(x[u]);
            run[0] += x[u];
            run[1] += it;
            run[2] += it > 1 ? it : 0u;
        }
        for (int q = 0; q < 3; ++q) {
            if (c + 4 <= m)
                *reinterpret_cast<uint4 *>(dst[q] + c) = make_uint4(o[q][0], o[q][1], o[q][2], o[q][3]);
            else
                for (int u = 0; u < 4 && c + u < m; ++u) dst[q][c + u] = o[q][u];
        }
    }
    if (threadIdx.x == 1023)  // (its candidates come last, or it has none: all sums)
        for (int q = 0; q < 3; ++q) dst[q][m] = run[q];
    if (threadIdx.x < OCC_QUEUES) a.tickets[threadIdx.x * TICKET_STRIDE] = 0u;
}

// Accumulation items: chunks of one candidate r's occurrences.  For an
// occurrence of r at position t of ballot v, every id ahead of it gains the
// voter's weight in the LDS row (C[id][r]), and r gains it in R.  PACKED
// (unit weights): two 16-bit counts per LDS word (an item adds at most
// OCC_CHUNK_MAX to a column).  The only item of a row writes the row of d
// (d[r][y] = base + R - C[y][r], base = full-ranking counts in acc or 0); an
// item of a heavier row writes its counts to its partial row and adds its
// part of R to rsum[r].
//
// Most candidates have few occurrences, so an item is a chain of dependent
// loads (item, occurrences, ballots) and then a row of d to write, with room
// for two to four LDS rows on a CU to hide them.  The workgroups stay: each
// starts with two items and draws the others from a queue per die (heavy
// candidates' items come in a run and fall to different workgroups), loads the
// next item's occurrences while it adds this one's ids and the next item's
// first ids while it writes this one's row, and clears the LDS row as it reads
// it out.  Ids come 16 bytes at a time at any alignment, as a scattered load
// costs its lane the same whatever its width.
//   m = 14187, 15553 ballots of 150 uint16 ids, half cut short:  508 -> 314 us
//   m = 16384, 1M ballots of 20 uint16 ids, int32 d:             547 -> 465
//   m = 32768, 200000 ballots of 30 uint16 ids, int32 d:        1434 -> 824
//   m = 6007, 100003 ballots of 12 int32 ids, int32 d:           110 -> 45
// (before: a workgroup per item, its row found by a binary search.)  Rows of
// d go out as streaming stores: through the caches the third took 1073.
//
// Ballots longer than the first pieces are read one occurrence after the
// other, the next pieces in flight while these are added.  Reading a thread's
// two occurrences side by side kept twice as many rows live in the L2, and
// with few wavefronts per CU (voter weights: 64 KB rows) nothing hid the wait
// for each step.  The whole count, us, with voter weights:
//                                        an id a load   side by side   so
//   m = 1500, 3000 up to 1500 int32 ids      2281           3470      1820
//   m = 1500, 3000 up to 1500 uint16 ids     2274           2500      1716
//   m = 5000, 30000 of 150 int32 ids          866           1065       685
//   m = 5000, 30000 of 25 int32 ids           197            169       166
constexpr int OCC_BATCH = 2, OCC_FLY = 4;  // occurrences per thread, pieces of ids of each in flight
template <int MAXM, bool PACKED, typename T, bool I32>
__global__ __launch_bounds__(256) void k_occ_accumulate(OccArgs a, T *__restrict__ d, int64_t ldd, uint32_t limit,
                                                        uint8_t *__restrict__ over_flag, int acc_zero) {
    constexpr int WORDS = PACKED ? MAXM / 2 : MAXM;
    __shared__ __attribute__((aligned(16))) uint32_t row[WORDS];
    __shared__ uint32_t wsum[2], ticket;
    if (a.meta.ctr[2] != MODE_SPARSE) return;
    const uint32_t total = __builtin_amdgcn_readfirstlane(a.item_start[a.m]), G = gridDim.x;
    if (blockIdx.x >= total) return;
    const int32_t m = a.m;
    const int32_t words = PACKED ? (m + 1) / 2 : m;
    const int32_t words4 = (words + 3) / 4;
    uint4 *row4 = reinterpret_cast<uint4 *>(row);
    for (int32_t c = threadIdx.x; c < words4; c += 256) row4[c] = make_uint4(0u, 0u, 0u, 0u);
    if (threadIdx.x < 2) wsum[threadIdx.x] = 0u;

    using Id = typename std::conditional<I32, int32_t, uint16_t>::type;
    constexpr int V = 16 / (int)sizeof(Id);  // ids per piece
    const Id *ids = static_cast<const Id *>(a.ballots);
    const int64_t last = a.n * a.L - V;  // the last piece inside the ballots (negative: less than a piece in all)
    const uint32_t tmask = (1u << a.tbits) - 1u;
    struct Item {
        uint32_t r, begin, end, partial;
    };
    auto item_of = [](const uint4 &q) {
        return Item{(uint32_t)__builtin_amdgcn_readfirstlane(q.x), (uint32_t)__builtin_amdgcn_readfirstlane(q.y),
                    (uint32_t)__builtin_amdgcn_readfirstlane(q.z), (uint32_t)__builtin_amdgcn_readfirstlane(q.w)};
    };
    // a thread's occurrences q and q + 256 of an item, and their first ids
    auto occ_in = [&](uint32_t (&ov)[OCC_BATCH], uint32_t q, uint32_t end) {
#pragma unroll
        for (int u = 0; u < OCC_BATCH; ++u) ov[u] = a.occ[min(q + 256 * u, end - 1)];
    };
    struct Occ {
        const Id *ids;  // the ballot
        int32_t t;      // position: so many ids are ahead
        int32_t lim;    // position of the last piece inside the ballots, at most 2^30
        uint32_t w;
    };
    Occ oc[OCC_BATCH];
    uint4 x[OCC_BATCH][OCC_FLY];
    auto piece = [&](const Occ &o, int32_t i) { return tio::load16<Id>(o.ids + min(i, o.lim)); };
    auto begin_ids = [&](const uint32_t (&ov)[OCC_BATCH], uint32_t q, uint32_t end) {
#pragma unroll
        for (int u = 0; u < OCC_BATCH; ++u) {
            const int64_t v = ov[u] >> a.tbits, b = v * a.L;
            oc[u].ids = ids + b;
            oc[u].lim = (int32_t)min(last - b, (int64_t)1 << 30);
            oc[u].w = q + 256 * u >= end ? 0u : (PACKED ? 1u : (a.weight ? a.weight[v] : 1u));
            oc[u].t = oc[u].w ? (int32_t)(ov[u] & tmask) : 0;
        }
#pragma unroll
        for (int u = 0; u < OCC_BATCH; ++u)
#pragma unroll
            for (int f = 0; f < OCC_FLY; ++f)
                if (V * f < oc[u].t && last >= 0) x[u][f] = piece(oc[u], V * f);
    };
    bool dup = false, over = false;
    uint32_t r = 0;
    auto add = [&](bool in, uint32_t id, uint32_t weight) {
        dup |= in && id == r;
        if (in && id < (uint32_t)m) {  // (not padding)
            if (PACKED)
                atomicAdd(&row[id >> 1], 1u << ((id & 1) * 16));
            else
                atomicAdd(&row[id], weight);
        }
    };
    // the ids at positions i .. of an occurrence, from their piece
    auto add_piece = [&](const Occ &o, int32_t i, const uint4 &xp) {
        if (i >= o.t) return;
        if (last < 0) {
            for (int32_t k = i; k < min(i + V, o.t); ++k) add(true, load_raw<I32>(o.ids, k), o.w);
            return;
        }
        // (the ballots' last piece may start before position i: skip to it)
        const int32_t skip = max(i - o.lim, 0), left = o.t - i;
        Id e[V];
        tio::unpack<Id>(xp, e);
#pragma unroll
        for (int k = 0; k < V; ++k) add((uint32_t)(k - skip) < (uint32_t)left, (uint32_t)e[k], o.w);
    };

    Item it = item_of(a.items[blockIdx.x]), next = item_of(a.items[min(blockIdx.x + G, total - 1)]);
    uint32_t ov[OCC_BATCH];
    occ_in(ov, it.begin + threadIdx.x, it.end);
    begin_ids(ov, it.begin + threadIdx.x, it.end);
    int parity = 0;
    uint32_t *queue = a.tickets + (blockIdx.x % OCC_QUEUES) * TICKET_STRIDE;
    uint32_t ahead = blockIdx.x + G;  // the next item's number
    for (uint32_t item = blockIdx.x; item < total; parity ^= 1) {
        occ_in(ov, next.begin + threadIdx.x, next.end);
        uint32_t drawn = 0;
        if (threadIdx.x == 0) drawn = atomicAdd(queue, 1u);
        __syncthreads();  // the LDS row is clear
        r = it.r;
        uint32_t wpart = 0;
        for (uint32_t q = it.begin + threadIdx.x;;) {
#pragma unroll
            for (int u = 0; u < OCC_BATCH; ++u) {
                wpart += oc[u].w;
#pragma unroll
                for (int f = 0; f < OCC_FLY; ++f) add_piece(oc[u], V * f, x[u][f]);
            }
            // the rest of longer ballots, one occurrence after the other
            constexpr int32_t STEP = V * OCC_FLY;
#pragma unroll 1
            for (int u = 0; u < OCC_BATCH; ++u) {
                Occ o = oc[0];
                if (u) o = oc[1];
                int32_t i = STEP;
                if (i >= o.t || last < 0) continue;
                auto pieces_in = [&](int h, int32_t at) {
#pragma unroll
                    for (int f = 0; f < OCC_FLY; ++f) x[h][f] = piece(o, at + V * f);
                };
                auto pieces_add = [&](int h) {
#pragma unroll
                    for (int f = 0; f < OCC_FLY; ++f) add_piece(o, i + V * f, x[h][f]);
                };
                pieces_in(0, i);
                if (o.t <= 2 * STEP) {
                    pieces_add(0);
                    continue;
                }
#pragma unroll 1
                for (;;) {  // the next pieces in flight while these are added
                    pieces_in(1, i + STEP);
                    pieces_add(0);
                    if ((i += STEP) >= o.t) break;
                    pieces_in(0, i + STEP);
                    pieces_add(1);
                    if ((i += STEP) >= o.t) break;
                }
            }
            q += 256 * OCC_BATCH;
            if (q >= it.end) break;
            uint32_t more[OCC_BATCH];
            occ_in(more, q, it.end);
            begin_ids(more, q, it.end);
        }
        if (!PACKED && wpart) atomicAdd(&wsum[parity], wpart);
        begin_ids(ov, next.begin + threadIdx.x, next.end);
        if (threadIdx.x == 0) ticket = 2 * G + blockIdx.x % OCC_QUEUES + OCC_QUEUES * drawn;
        __syncthreads();
        item = ahead;
        ahead = ticket;  // (written again only after the next barrier)
        const uint4 after = a.items[min(ahead, total - 1)];
        const uint32_t R = PACKED ? it.end - it.begin : wsum[parity];
        if (threadIdx.x == 0) wsum[parity ^ 1] = 0u;
        if (it.partial == NO_PARTIAL) {
            // the row's only item: d[r][y] = base + R - C[y][r]; the finish skips the row
            const uint32_t *arow = a.acc + (int64_t)r * a.lda;
            T *drow = d + (int64_t)r * ldd;
            constexpr int C = 16 / (int)sizeof(T);         // columns per store
            constexpr int CW = PACKED ? C / 2 : C;         // their LDS words
            auto value = [&](uint32_t cnt, uint32_t full, int32_t y) -> uint32_t {
                const uint32_t v = y == (int32_t)r ? 0u : full - cnt + R;
                over |= v > limit;
                return min(v, limit);
            };
            for (int32_t y = C * threadIdx.x; y < m; y += C * 256) {
                uint32_t cw[CW];
                uint32_t *rw = row + (PACKED ? y / 2 : y);
                if (y + C <= m) {
#pragma unroll
                    for (int k = 0; k < CW; ++k) cw[k] = rw[k];
#pragma unroll
                    for (int k = 0; k < CW; ++k) rw[k] = 0u;
                    T o[C];
#pragma unroll
                    for (int k = 0; k < C; ++k) {
                        const uint32_t cnt = PACKED ? (cw[k / 2] >> (16 * (k & 1))) & 0xFFFFu : cw[k % CW];
                        o[k] = (T)value(cnt, acc_zero ? 0u : arow[y + k], y + k);
                    }
                    tio::stream16<T>(drow + y, tio::pack<T>(o));
                } else {
                    for (int32_t yy = y; yy < m; ++yy) {
                        const uint32_t cnt = PACKED ? (row[yy >> 1] >> ((yy & 1) * 16)) & 0xFFFFu : row[yy];
                        drow[yy] = (T)value(cnt, acc_zero ? 0u : arow[yy], yy);
                    }
                    for (int32_t k = 0; k < (PACKED ? (m - y + 1) / 2 : m - y); ++k) rw[k] = 0u;
                }
            }
        } else {
            // an item of a heavier row: its partial row (same element layout as the LDS row)
            uint4 *prow = reinterpret_cast<uint4 *>(static_cast<uint32_t *>(a.partial) +
                                                    (int64_t)it.partial * (a.ppitch * (PACKED ? 1 : 2) / 2));
            for (int32_t c = threadIdx.x; c < words4; c += 256) {
                prow[c] = row4[c];
                row4[c] = make_uint4(0u, 0u, 0u, 0u);
            }
            if (threadIdx.x == 0 && R) atomicAdd(&a.rsum[r], R);
        }
        it = next;
        next = item_of(after);
    }
    if (__ballot(dup) && (threadIdx.x & 63) == 0) set_device_error(a.err, SCHULZE_EBALLOT);
    // reported by the finish, after every ballot error of this launch
    if (over) over_flag[0] = 1;
}

// Rows the accumulation items did not finish: candidates without
// occurrences (d[r][y] = base) and heavier candidates (d[r][y] = base + R_r
// - sum of their partial rows), as listed by the column pass.  Persistent:
// units (listed row, block of OCC_FIN_COLS columns) dealt to the
// workgroups in turn (a walk over every row that skipped the finished ones
// waited for memory at each); a thread takes eight consecutive columns (one
// 16-byte read per partial row of unit weights), four partial rows in
// flight.  Also reports an overflow found by the accumulation.
template <typename T, bool PACKED>
__global__ __launch_bounds__(256) void k_occ_finish(OccArgs a, T *__restrict__ d, int64_t ldd, uint32_t limit,
                                                    const uint8_t *__restrict__ over_flag, int acc_zero) {
    static_assert(OCC_FIN_COLS == 8 * 256, "a thread takes eight columns");
    if (a.meta.ctr[2] != MODE_SPARSE) return;
    const int32_t m = a.m;
    if (blockIdx.x == 0 && threadIdx.x == 0 && over_flag[0]) set_device_error(a.err, SCHULZE_ERANGE);
    const int32_t cb = (m + OCC_FIN_COLS - 1) / OCC_FIN_COLS;
    const bool avec = (a.lda % 4) == 0;  // rows of acc 16-byte aligned
    const int32_t nfin = a.meta.ctr[FIN_COUNT];
    bool over = false;
    for (int64_t u = blockIdx.x; u < (int64_t)nfin * cb; u += gridDim.x) {
        const int32_t r = a.fin[u / cb];
        const int32_t y = (int32_t)(u % cb) * OCC_FIN_COLS + 8 * threadIdx.x;
        if (y >= m) continue;
        const uint32_t p0 = a.part_start[r], np = a.part_start[r + 1] - p0;
        const uint32_t R = np ? a.rsum[r] : 0u;
        uint32_t c[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
        // partial rows hold round_up(m, 8) columns: eight at y are always there
        auto add_row = [&](uint32_t k) {
            const int64_t off = (int64_t)(p0 + k) * a.ppitch + y;
            if constexpr (PACKED) {
                const uint4 x = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(a.partial) + off);
                const uint32_t w[4] = {x.x, x.y, x.z, x.w};
                for (int e = 0; e < 4; ++e) {
                    c[2 * e] += w[e] & 0xFFFFu;
                    c[2 * e + 1] += w[e] >> 16;
                }
            } else {
                const uint4 *q = reinterpret_cast<const uint4 *>(static_cast<const uint32_t *>(a.partial) + off);
                const uint4 x0 = q[0], x1 = q[1];
                c[0] += x0.x, c[1] += x0.y, c[2] += x0.z, c[3] += x0.w;
                c[4] += x1.x, c[5] += x1.y, c[6] += x1.z, c[7] += x1.w;
            }
        };
        uint32_t k = 0;
        for (; k + 4 <= np; k += 4) {
            add_row(k);
            add_row(k + 1);
            add_row(k + 2);
            add_row(k + 3);
        }
        for (; k < np; ++k) add_row(k);
        uint32_t base[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
        if (!acc_zero) {
            const uint32_t *arow = a.acc + (int64_t)r * a.lda;
            if (avec && y + 8 <= m) {
                const uint4 b0 = *reinterpret_cast<const uint4 *>(arow + y), b1 = *reinterpret_cast<const uint4 *>(arow + y + 4);
                base[0] = b0.x, base[1] = b0.y, base[2] = b0.z, base[3] = b0.w;
                base[4] = b1.x, base[5] = b1.y, base[6] = b1.z, base[7] = b1.w;
            } else {
                for (int e = 0; e < 8 && y + e < m; ++e) base[e] = arow[y + e];
            }
        }
        uint32_t v[8];
        for (int e = 0; e < 8; ++e) {
            v[e] = y + e == r ? 0u : base[e] - c[e] + R;
            // (columns past m: the partial rows of 32-bit counts are written up to a multiple of 4 only)
            if (v[e] > limit && y + e < m) {
                over = true;
                v[e] = limit;
            }
        }
        store8<T>(d + (int64_t)r * ldd, y, m, v);
    }
    if (over) set_device_error(a.err, SCHULZE_ERANGE);
}

// ------------------------------------------------------------------ finish
// d[x][y] = acc[x][y] plus the truncated ballots' R term, 0 on the
// diagonal; range-checked store.
template <typename T>
__global__ __launch_bounds__(256) void k_count_finish(const uint32_t *__restrict__ acc, int64_t lda,
                                                      const uint32_t *__restrict__ rsum, Meta meta, int32_t m,
                                                      T *__restrict__ d, int64_t ldd, uint32_t limit, int32_t *err,
                                                      int bucketed) {
    // one workgroup per row x; the bucketed route writes its own rows
    const int32_t x = blockIdx.x;
    if (bucketed && meta.ctr[2] == MODE_SPARSE) return;
    const bool dense_u = meta.ctr[2] == MODE_DENSE_U;
    const uint32_t rx = rsum[x];
    const bool in_x = dense_u && meta.in_u[x];
    bool over = false;
    for (int32_t y = threadIdx.x; y < m; y += 256) {
        uint32_t v = 0u;
        if (x != y) {
            v = acc[(int64_t)x * lda + y];
            // pair scattering: acc holds -C^T, add R[x]; dense over U: U x U is
            // complete, x in U beats every y outside U on the R[x] ballots
            if (!dense_u || (in_x && !meta.in_u[y])) v += rx;
        }
        if (v > limit) {
            over = true;
            v = limit;
        }
        d[(int64_t)x * ldd + y] = (T)v;
    }
    if (over) set_device_error(err, SCHULZE_ERANGE);
}

// Byte layout of WS_BALLOT_META for n ballots and m candidates.
// Total voter weight in 64 bits: counts accumulate in 32-bit words, which
// cannot wrap while the total stays below 2^32 (and then the finish checks
// every count against the value type); a total of 2^32 or more sets
// SCHULZE_ERANGE.  total and done start at zero; the last workgroup to add
// its part decides, and then passes on an error recorded in *later, which a
// profile with both is to report second (nullptr: none).
__global__ __launch_bounds__(256) void k_weight_total(const uint32_t *__restrict__ w, int64_t n,
                                                      unsigned long long *total, int32_t *done, int32_t *any,
                                                      const int32_t *later, int32_t *err) {
    __shared__ unsigned long long part[256];
    unsigned long long acc = 0;
    uint32_t ored = 0u;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        acc += w[i];
        ored |= w[i];
    }
    for (int off = 32; off >= 1; off >>= 1) ored |= __shfl_xor(ored, off);
    if ((threadIdx.x & 63) == 0 && ored) atomicOr(any, (int32_t)ored);
    part[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) part[threadIdx.x] += part[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        atomicAdd(total, part[0]);
        __threadfence();
        if (atomicAdd(done, 1) == (int32_t)gridDim.x - 1) {
            __threadfence();
            if (atomicAdd(total, 0ull) >> 32) set_device_error(err, SCHULZE_ERANGE);
            if (later && *later != 0) set_device_error(err, *later);
        }
    }
}

// Zero the m x m accumulator, unless skip_bucketed and the device chose the
// bucketed route (which then does not read it).
__global__ __launch_bounds__(256) void k_fill_acc(uint32_t *__restrict__ p, int64_t words, Meta meta,
                                                  int skip_bucketed) {
    if (skip_bucketed && meta.ctr[2] == MODE_SPARSE) return;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, stride = (int64_t)gridDim.x * 256;
    uint4 *p4 = reinterpret_cast<uint4 *>(p);  // workspace: 16-byte aligned
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    for (int64_t j = i; j < words / 4; j += stride) p4[j] = z;
    for (int64_t j = words / 4 * 4 + i; j < words; j += stride) p[j] = 0u;
}

struct MetaLayout {
    // cleared by each call: ctr .. rsum (one fill); then the rest
    size_t ctr, k2, over, in_u, rsum, len, full_src, trunc_src, ulist, umap, total;
    MetaLayout(int64_t n, int32_t m) {
        size_t o = 0;
        auto take = [&](size_t bytes) {
            size_t at = o;
            o += (bytes + 255) / 256 * 256;
            return at;
        };
        ctr = take(64 * sizeof(int32_t));
        k2 = take(NPART * sizeof(unsigned long long));
        over = take(sizeof(uint32_t));  // a count above the limit was clamped (bucketed route)
        in_u = take((size_t)m);
        rsum = take(sizeof(uint32_t) * (size_t)m);
        len = take(sizeof(int32_t) * (size_t)n);
        full_src = take(sizeof(int32_t) * (size_t)n);
        trunc_src = take(sizeof(int32_t) * (size_t)n);
        ulist = take(sizeof(int32_t) * (size_t)m);
        umap = take(sizeof(int32_t) * (size_t)m);
        total = o;
    }
};

// Byte layout of WS_OCC for G bucketing workgroups, m candidates and at
// most cap occurrences.
// Partial rows: every item of a candidate with two or more items has one,
// and such a candidate has more than a chunk of occurrences, so there are at
// most 2 cap / chunk of them.
struct OccLayout {
    size_t hist, row_start, items, item_start, tickets, part_start, fin, occ, partial, total;
    int64_t ppitch, max_parts;
    uint32_t chunk;  // occurrences per accumulation item, of at most cap, for this many workgroups
    OccLayout(int64_t G, int32_t m, int64_t cap, size_t partial_elem, int64_t workgroups) {
        size_t o = 0;
        auto take = [&](size_t bytes) {
            size_t at = o;
            o += (bytes + 255) / 256 * 256;
            return at;
        };
        ppitch = round_up(m, 8);
        chunk = (uint32_t)std::min<int64_t>(OCC_CHUNK_MAX, std::max<int64_t>(OCC_CHUNK_MIN, cap / (4 * workgroups)));
        // room for ceil(cap / chunk) chunks, by a bound that never falls as cap
        // grows: up to the smallest chunk's, then about 4 per workgroup, then
        // the largest chunk's
        const int64_t chunks = std::min(ceil_div(cap, OCC_CHUNK_MIN),
                                        std::max(4 * workgroups + 4 * workgroups / OCC_CHUNK_MIN + 2,
                                                 ceil_div(cap, OCC_CHUNK_MAX)));
        max_parts = cap > 0 ? 2 * chunks + 1 : 0;
        hist = take(sizeof(uint32_t) * (size_t)G * m);
        row_start = take(sizeof(uint32_t) * ((size_t)m + 1));
        items = take(sizeof(uint4) * ((size_t)m + (size_t)chunks));
        item_start = take(sizeof(uint32_t) * ((size_t)m + 1));
        tickets = take(sizeof(uint32_t) * OCC_QUEUES * TICKET_STRIDE);
        part_start = take(sizeof(uint32_t) * ((size_t)m + 1));
        occ = take(sizeof(uint32_t) * (size_t)cap);
        partial = take(partial_elem * (size_t)max_parts * (size_t)ppitch);
        fin = take(sizeof(int32_t) * (size_t)m);
        total = o;
    }
};

// The counting (PLACE = false) or placing pass of the bucketing, for the LDS
// histogram that fits m and the ballots' id type.
template <bool PLACE>
int occ_bucket(schulze_ctx *ctx, hipStream_t s, const OccArgs &oa, dim3 g) {
    const dim3 b(256);
    if (oa.m <= OCC_MAX_M / 2) {
        if (oa.dtype32)
            SCHULZE_LAUNCH(ctx, K_COUNT_SPARSE, s, (k_occ_bucket<OCC_MAX_M / 2, PLACE, true><<<g, b, 0, s>>>(oa)));
        else
            SCHULZE_LAUNCH(ctx, K_COUNT_SPARSE, s, (k_occ_bucket<OCC_MAX_M / 2, PLACE, false><<<g, b, 0, s>>>(oa)));
    } else {
        if (oa.dtype32)
            SCHULZE_LAUNCH(ctx, K_COUNT_SPARSE, s, (k_occ_bucket<OCC_MAX_M, PLACE, true><<<g, b, 0, s>>>(oa)));
        else
            SCHULZE_LAUNCH(ctx, K_COUNT_SPARSE, s, (k_occ_bucket<OCC_MAX_M, PLACE, false><<<g, b, 0, s>>>(oa)));
    }
    return SCHULZE_OK;
}

// The accumulation and finish launches for the counter type T of d: packed
// 16-bit LDS counts for unit weights, 32-bit ones otherwise; the LDS row fits
// m.
template <typename T, int MAXM, bool PACKED>
int occ_accumulate_m(schulze_ctx *ctx, hipStream_t s, const OccArgs &oa, dim3 grid, T *d, int64_t ldd,
                     uint32_t limit, uint8_t *over_flag, int az) {
    const dim3 b(256);
    if (oa.dtype32)
        SCHULZE_LAUNCH(ctx, K_COUNT_SPARSE, s,
                       (k_occ_accumulate<MAXM, PACKED, T, true><<<grid, b, 0, s>>>(oa, d, ldd, limit, over_flag, az)));
    else
        SCHULZE_LAUNCH(ctx, K_COUNT_SPARSE, s,
                       (k_occ_accumulate<MAXM, PACKED, T, false><<<grid, b, 0, s>>>(oa, d, ldd, limit, over_flag, az)));
    return SCHULZE_OK;
}

template <typename T>
int occ_accumulate(schulze_ctx *ctx, hipStream_t s, const OccArgs &oa, dim3 grid, int32_t m, bool weighted, T *d,
                   int64_t ldd, uint32_t limit, uint8_t *over_flag, bool acc_zero) {
    const int az = acc_zero ? 1 : 0;
    int rc;
    if (!weighted && m <= OCC_MAX_M / 2)
        rc = occ_accumulate_m<T, OCC_MAX_M / 2, true>(ctx, s, oa, grid, d, ldd, limit, over_flag, az);
    else if (!weighted)
        rc = occ_accumulate_m<T, OCC_MAX_M, true>(ctx, s, oa, grid, d, ldd, limit, over_flag, az);
    else if (m <= OCC_MAX_M / 2)
        rc = occ_accumulate_m<T, OCC_MAX_M / 2, false>(ctx, s, oa, grid, d, ldd, limit, over_flag, az);
    else
        rc = occ_accumulate_m<T, OCC_MAX_M, false>(ctx, s, oa, grid, d, ldd, limit, over_flag, az);
    if (rc != SCHULZE_OK) return rc;
    const dim3 fg((unsigned)(ctx->num_cus * 4));
    if (weighted) {
        SCHULZE_LAUNCH(ctx, K_COUNT_FINISH, s,
                       (k_occ_finish<T, false><<<fg, dim3(256), 0, s>>>(oa, d, ldd, limit, over_flag, az)));
    } else {
        SCHULZE_LAUNCH(ctx, K_COUNT_FINISH, s,
                       (k_occ_finish<T, true><<<fg, dim3(256), 0, s>>>(oa, d, ldd, limit, over_flag, az)));
    }
    return SCHULZE_OK;
}

// The total voter weight (counters 32 and 33, and the workgroups done in 34)
// and the weights or-ed (7); all start at zero.  later: see k_weight_total.
int weight_total(schulze_ctx *ctx, hipStream_t s, const uint32_t *weight, int64_t n, int32_t *ctr,
                 const int32_t *later = nullptr) {
    const unsigned tg = (unsigned)std::min<int64_t>(ceil_div(n, 256), (int64_t)ctx->num_cus * 4);
    SCHULZE_LAUNCH(ctx, K_ROUTE, s,
                   k_weight_total<<<dim3(tg), dim3(256), 0, s>>>(weight, n, reinterpret_cast<unsigned long long *>(ctr + 32),
                                                                 ctr + 34, ctr + 7, later, ctx->err));
    return SCHULZE_OK;
}

// Rank planes and the bit-plane count of the full rankings (FULL) or, if the
// device chose the dense route, of the truncated ballots over U (pitch: at
// most that many columns).  A workgroup of the planes takes 2048 columns
// with 1024 threads (128 KB of LDS; each further chunk of columns reads the
// ballots again) or, for at most 1024 columns, 512 with 256 threads.
template <bool FULL>
int count_dense(schulze_ctx *ctx, hipStream_t s, const void *ballots, int dtype32, int64_t n, int32_t L, int32_t m, int32_t pitch,
                int32_t bits, int64_t max_groups, const Meta &meta, const uint32_t *weight, uint32_t *planes,
                uint32_t *wplanes, uint32_t *acc, int64_t lda, uint32_t *rsum) {
    const PlaneArgs pa{ballots, L, m, pitch, bits, meta, weight, planes, wplanes, ctx->err, n};
    const int wide = pitch > 1024;
    // (the route may leave nothing to do: no more workgroups than stay resident)
    const dim3 pg((unsigned)std::min<int64_t>(max_groups * ceil_div(pitch, wide ? 2048 : 512),
                                              (int64_t)ctx->num_cus * (wide ? 1 : 4)));
    if (wide && dtype32)
        SCHULZE_LAUNCH(ctx, K_BALLOT_SCATTER, s, (k_planes<FULL, true, 2048, 1024><<<pg, dim3(1024), 0, s>>>(pa)));
    else if (wide)
        SCHULZE_LAUNCH(ctx, K_BALLOT_SCATTER, s, (k_planes<FULL, false, 2048, 1024><<<pg, dim3(1024), 0, s>>>(pa)));
    else if (dtype32)
        SCHULZE_LAUNCH(ctx, K_BALLOT_SCATTER, s, (k_planes<FULL, true, 512, 256><<<pg, dim3(256), 0, s>>>(pa)));
    else
        SCHULZE_LAUNCH(ctx, K_BALLOT_SCATTER, s, (k_planes<FULL, false, 512, 256><<<pg, dim3(256), 0, s>>>(pa)));
    const int32_t grid = ctx->num_cus * COUNT_PER_CU;
    DenseArgs da{};
    da.planes = planes, da.pitch = pitch, da.bits = bits, da.m = m, da.meta = meta;
    da.acc = acc, da.lda = lda, da.rsum = rsum, da.wplanes = wplanes;
    da.partial = static_cast<uint32_t *>(ctx->ws[WS_OCC]);
    const dim3 cg((unsigned)grid), rg((unsigned)std::min<int64_t>(64 * ceil_div(pitch, CT) * ceil_div(pitch, CT),
                                                                   (int64_t)ctx->num_cus * 8));
    const int kid = FULL ? K_COUNT_DENSE : K_COUNT_TRUNC;
    constexpr int MODE = FULL ? COUNT_FULL : COUNT_U;
    if (FULL && weight) {
        SCHULZE_LAUNCH(ctx, kid, s, (k_count_bits<MODE, FULL><<<cg, dim3(256), 0, s>>>(da)));
        SCHULZE_LAUNCH(ctx, kid, s, (k_count_reduce<MODE, FULL><<<rg, dim3(256), 0, s>>>(da, grid)));
    } else {
        SCHULZE_LAUNCH(ctx, kid, s, (k_count_bits<MODE, false><<<cg, dim3(256), 0, s>>>(da)));
        SCHULZE_LAUNCH(ctx, kid, s, (k_count_reduce<MODE, false><<<rg, dim3(256), 0, s>>>(da, grid)));
    }
    return SCHULZE_OK;
}

// Small elections: every ballot over all candidates in one dense pass, three
// launches (planes, count, adding up; five with voter weights) instead of the
// scan, the route decision and both routes' kernels (19, at about 4.5 us
// each even where they find nothing to do).  Taken while the count costs at
// most ALL_COST lane operations (65 us at 45 T/s), about what the other
// launches would.
//
// Voter weights cost some operations more per mask (weight_ops), and how many
// bits they have only the device knows.  Twelve planes' are charged against
// ALL_COST; but short ballots cost the routed count little more than its
// launches, so there the count has to win with as many bits as a total weight
// below 2^32 allows, 33 - log2(groups) on average.  In lane operations at 37 T/s
// the routed count is taken as 34 us (WIDE_COST; the rest of its 70 us is what
// the one pass launches too), 1.3 ps a cell of the matrix, 8 ns a ballot and 3
// ps for each pair that ballots of this length can list.  Counts in us, with
// weights of 6, 16 and 32 bits (at most: their total is below 2^32):
//                                one pass     by pairs   taken
//   m = 1000, n =  480, top-20   53  57  69      80      one pass
//   m = 1000, n = 1400, top-20   72  84 108      84      by pairs
//   m =  389, n = 7001, top-25   77  93 115      85      one pass
//   m =  128, n = 1e5,  top-10  104 117 118     130      one pass
//   m = 2000, n =  300, top-30   66  77 107      87      by pairs
//   m = 4096, n =   64, top-50   56  65  92     100      one pass
//   m = 1000, n = 1400, up to 1000 places
//                                82  94 118   92 to 700  one pass (92: all of them list 20)
constexpr int REPEATED = 9;  // counter that holds SCHULZE_EBALLOT if a ballot lists an id twice
constexpr double ALL_COST = 3.0e9;
constexpr double WIDE_COST = 1.25e9, ROUTED_CELL_COST = 50.0, ROUTED_BALLOT_COST = 3.1e5, LISTED_PAIR_COST = 112.0;
constexpr int32_t ALL_MAX_M = 4096;
inline bool count_all_fits(int64_t n, int32_t L, int32_t m, bool weighted) {
    if (n < 1 || m > ALL_MAX_M) return false;
    const int64_t groups = ceil_div(n, 32);
    const double pitch = (double)round_up(m, CT), work = (double)groups * pitch * pitch;
    const int32_t ops = rank_bits(std::min(L, m - 1)) + 2;
    if (work * (ops + (weighted ? 36 : 0)) > ALL_COST) return false;
    if (!weighted) return true;
    const int32_t bits = std::min(32, __builtin_clzll((uint64_t)groups) - 30);  // 33 - log2(groups)
    return work * (ops + weight_ops(bits)) <= WIDE_COST + ROUTED_CELL_COST * m * m + ROUTED_BALLOT_COST * n +
                                                  LISTED_PAIR_COST * 0.5 * (double)n * L * (L - 1);
}

// Workspace of the one-pass count (in WS_OCC): partial tiles, planes, planes
// of the weights.  Every part grows with n, L and m, so that the layout of a
// call holds every smaller one's.
struct AllLayout {
    int64_t groups, ntiles, workers;
    int32_t pitch, bits;
    bool whole;  // whole tiles per workgroup; else ranges of two units or more, whose partial tiles are added up
    size_t planes, wplanes, total;
    AllLayout(int64_t num_cus, int64_t n, int32_t L, int32_t m, bool weighted) {
        pitch = (int32_t)round_up(m, CT), bits = rank_bits(std::min(L, m - 1));
        groups = ceil_div(n, 32), ntiles = (int64_t)(pitch / CT) * (pitch / CT);
        const int64_t grid_max = num_cus * COUNT_PER_CU, ranges = std::min(grid_max, ceil_div(ntiles * groups, 2));
        whole = 2 * ntiles >= grid_max || groups == 1;
        workers = whole ? std::min(grid_max, ntiles) : ranges;
        // (unused when whole, but a smaller call may not be)
        const int64_t tiles = groups > 1 ? ranges + std::min(ntiles, grid_max / 2) : 0;
        // a call this large may be routed, but what ALL_COST lets through has at most ALL_COST / CT words of planes
        const size_t words = (size_t)std::min<double>((double)groups * bits * pitch, ALL_COST / CT);
        const size_t wwords = weighted ? WEIGHT_WORDS * (size_t)std::min<double>((double)groups, ALL_COST / (CT * CT)) : 0;
        planes = sizeof(uint32_t) * CT * CT * (size_t)tiles;
        wplanes = planes + sizeof(uint32_t) * words;
        total = wplanes + sizeof(uint32_t) * wwords;
    }
};

int count_all(schulze_ctx *ctx, hipStream_t s, const void *ballots, int dtype32, int64_t n, int32_t L, int32_t m,
              const uint32_t *weight, int d_dtype, void *d, int64_t ldd) {
    const AllLayout al(ctx->num_cus, n, L, m, weight != nullptr);
    const int32_t pitch = al.pitch, bits = al.bits;
    const int64_t groups = al.groups, ntiles = al.ntiles, workers = al.workers;
    const bool whole = al.whole;
    int rc = ws_reserve(ctx, WS_OCC, al.total);
    if (rc != SCHULZE_OK) return rc;
    if (weight && (rc = ws_reserve(ctx, WS_BALLOT_META, 64 * sizeof(int32_t))) != SCHULZE_OK) return rc;
    char *base = static_cast<char *>(ctx->ws[WS_OCC]);
    uint32_t *planes = reinterpret_cast<uint32_t *>(base + al.planes);
    DenseArgs da{};
    da.planes = planes, da.pitch = pitch, da.bits = bits, da.m = m;
    da.wplanes = weight ? reinterpret_cast<uint32_t *>(base + al.wplanes) : nullptr;
    da.partial = reinterpret_cast<uint32_t *>(base);
    da.n = (int32_t)n, da.whole = whole;
    da.d = d, da.ldd = ldd, da.d32 = d_dtype == SCHULZE_I32, da.err = ctx->err;
    da.limit = d_dtype == SCHULZE_U16 ? 65535u : (uint32_t)INT32_MAX;
    if (weight) {
        da.meta.ctr = static_cast<int32_t *>(ctx->ws[WS_BALLOT_META]);
        if ((rc = fill_u32(ctx, s, reinterpret_cast<uint32_t *>(da.meta.ctr), 64, 0u)) != SCHULZE_OK) return rc;
    }
    // the first error of a profile with several: an id out of range, a total
    // weight out of range, a repeated id, a count out of range (as the other routes')
    int32_t *repeated = weight ? da.meta.ctr + REPEATED : ctx->err;
    const AllArgs pa{ballots, (int32_t)n, L, m, pitch, bits, weight, planes, const_cast<uint32_t *>(da.wplanes), ctx->err,
                     repeated};
    rc = weight ? (dtype32 ? planes_all<true, true>(ctx, s, pa, groups) : planes_all<false, true>(ctx, s, pa, groups))
                : (dtype32 ? planes_all<true, false>(ctx, s, pa, groups) : planes_all<false, false>(ctx, s, pa, groups));
    if (rc != SCHULZE_OK) return rc;
    if (weight && (rc = weight_total(ctx, s, weight, n, da.meta.ctr, repeated)) != SCHULZE_OK) return rc;
    const dim3 cg((unsigned)workers), rg((unsigned)std::min<int64_t>(64 * ntiles, (int64_t)ctx->num_cus * 8));
    if (weight)
        SCHULZE_LAUNCH(ctx, K_COUNT_DENSE, s, (k_count_bits<COUNT_ALL, true><<<cg, dim3(256), 0, s>>>(da)));
    else
        SCHULZE_LAUNCH(ctx, K_COUNT_DENSE, s, (k_count_bits<COUNT_ALL, false><<<cg, dim3(256), 0, s>>>(da)));
    if (!whole)
        SCHULZE_LAUNCH(ctx, K_COUNT_FINISH, s,
                       (k_count_reduce<COUNT_ALL, false><<<rg, dim3(256), 0, s>>>(da, (int32_t)workers)));
    return SCHULZE_OK;
}

constexpr size_t TRUNC_PLANES_CAP = (size_t)1 << 30;

}  // namespace

extern "C" int schulze_pairwise(schulze_ctx *ctx, void *stream, const void *ballots, int ballot_dtype, int64_t n,
                                int32_t L, int32_t m, const uint32_t *voter_weight, int d_dtype, void *d,
                                int64_t ldd) {
    if (!ctx || !d) return SCHULZE_EINVAL;
    if (ballot_dtype != SCHULZE_U16 && ballot_dtype != SCHULZE_I32) return SCHULZE_EINVAL;
    if (d_dtype != SCHULZE_U16 && d_dtype != SCHULZE_I32) return SCHULZE_EINVAL;
    if (n < 0 || m < 1 || m > 65535 || L < 1 || L > m || ldd < m) return SCHULZE_EINVAL;
    if (n > 0 && !ballots) return SCHULZE_EINVAL;
    if (n > (int64_t)INT32_MAX) return SCHULZE_EUNSUPPORTED;
    if (d_dtype == SCHULZE_U16 && !voter_weight && n > 65535) return SCHULZE_ERANGE;
    if (bind_device(ctx) != SCHULZE_OK) return SCHULZE_EDEVICE;
    hipStream_t s = (hipStream_t)stream;
    const int dtype32 = ballot_dtype == SCHULZE_I32;
    const bool one_pass = !ctx->legacy_pairs && count_all_fits(n, L, m, voter_weight != nullptr);
    if (one_pass && !voter_weight) return count_all(ctx, s, ballots, dtype32, n, L, m, nullptr, d_dtype, d, ldd);
    const int32_t pitch = (int32_t)round_up(m, CT);
    const int64_t max_groups = ceil_div(n, 32);  // of 32 voters
    const bool may_have_full = L >= m - 1 && n > 0;
    const bool may_have_trunc = n > 0;  // a row may always end early
    const int64_t upitch_max = round_up((int64_t)m + 1, CT);
    const int32_t full_bits = rank_bits(m - 1), trunc_bits = rank_bits(L);
    const size_t trunc_bytes =
        may_have_trunc && !voter_weight
            ? std::min(TRUNC_PLANES_CAP,
                       sizeof(uint32_t) * (size_t)max_groups * trunc_bits * (size_t)upitch_max)
            : 0;
    // weights: planes per group of the full rankings (weighted truncated ballots are counted by pairs)
    const size_t weight_words = voter_weight ? WEIGHT_WORDS * (size_t)max_groups : 0;

    const MetaLayout lay(n, m);
    int rc;
    if ((rc = ws_reserve(ctx, WS_BALLOT_META, lay.total)) != SCHULZE_OK) return rc;
    if ((rc = ws_reserve(ctx, WS_ACC32, sizeof(uint32_t) * (size_t)m * m)) != SCHULZE_OK) return rc;
    if (may_have_full &&
        (rc = ws_reserve(ctx, WS_POSITIONS, sizeof(uint32_t) * ((size_t)max_groups * full_bits * pitch + weight_words))) !=
            SCHULZE_OK)
        return rc;
    if (trunc_bytes &&
        (rc = ws_reserve(ctx, WS_TRUNC_POS, trunc_bytes)) != SCHULZE_OK)
        return rc;
    // bucketed pair counting: an LDS row of counts per candidate and a bounded occurrence buffer
    const int64_t occ_cap = n * (int64_t)L;
    const bool occ_ok = n > 0 && m <= OCC_MAX_M && occ_cap <= OCC_MAX && !ctx->legacy_pairs;
    const int64_t occ_grid = (int64_t)ctx->num_cus * (m <= OCC_MAX_M / 2 ? 2 : 1);
    // as many accumulation workgroups as LDS rows fit the CUs (160 KB each; at most four by registers)
    const int64_t acc_row = (m <= OCC_MAX_M / 2 ? OCC_MAX_M / 2 : OCC_MAX_M) * (voter_weight ? 4 : 2) + 256;
    const int64_t acc_grid = ctx->num_cus * std::min<int64_t>(4, 160 * 1024 / acc_row);
    const OccLayout ol(occ_ok ? occ_grid : 0, m, occ_ok ? occ_cap : 0, voter_weight ? 4 : 2, acc_grid);
    // the same memory in turn: the dense counts' partial tiles, then the
    // bucketed count's, and in a smaller call all of the one-pass count's
    const size_t scratch = std::max({sizeof(uint32_t) * 2 * CT * CT * (size_t)ctx->num_cus * COUNT_PER_CU,
                                     occ_ok ? ol.total : 0, AllLayout(ctx->num_cus, n, L, m, voter_weight != nullptr).total});
    if (n > 0 && (rc = ws_reserve(ctx, WS_OCC, scratch)) != SCHULZE_OK) return rc;
    // (after the reservations: with weights a smaller call may be routed)
    if (one_pass) return count_all(ctx, s, ballots, dtype32, n, L, m, voter_weight, d_dtype, d, ldd);

    char *mb = static_cast<char *>(ctx->ws[WS_BALLOT_META]);
    Meta meta{reinterpret_cast<int32_t *>(mb + lay.ctr),
              reinterpret_cast<unsigned long long *>(mb + lay.k2),
              reinterpret_cast<int32_t *>(mb + lay.len),
              reinterpret_cast<int32_t *>(mb + lay.full_src),
              reinterpret_cast<int32_t *>(mb + lay.trunc_src),
              reinterpret_cast<uint8_t *>(mb + lay.in_u),
              reinterpret_cast<int32_t *>(mb + lay.ulist),
              reinterpret_cast<int32_t *>(mb + lay.umap)};
    uint32_t *acc = static_cast<uint32_t *>(ctx->ws[WS_ACC32]);
    uint32_t *rsum = reinterpret_cast<uint32_t *>(mb + lay.rsum);
    const int64_t lda = m;

    // counters, partial sums, the U bitmap and the row sums start at zero
    if ((rc = fill_u32(ctx, s, reinterpret_cast<uint32_t *>(mb), lay.len / 4, 0u)) != SCHULZE_OK) return rc;
    if (n == 0 && (rc = fill_u32(ctx, s, acc, (size_t)m * m, 0u)) != SCHULZE_OK) return rc;

    uint8_t *over_flag = nullptr;  // the bucketed count's overflow flag (set: it ran and wrote its rows)
    if (n > 0) {
        if (L <= 64) {
            // more ballots per workgroup where there are many (fewer reservations)
            const int64_t per_round = 4 * SHORT_PER_WAVE * std::min<int64_t>(SHORT_BPW, 64 / L);
            const int32_t rounds = (int32_t)std::max<int64_t>(
                SHORT_ROUNDS, std::min<int64_t>(SHORT_MAX_ROUNDS, ceil_div(n, per_round * 2 * ctx->num_cus)));
            const dim3 sg((unsigned)ceil_div(n, per_round * rounds));
            if (dtype32)
                SCHULZE_LAUNCH(ctx, K_BALLOT_SCAN, s,
                               k_scan_short<true><<<sg, dim3(256), 0, s>>>(ballots, n, L, m, rounds, meta, ctx->err));
            else
                SCHULZE_LAUNCH(ctx, K_BALLOT_SCAN, s,
                               k_scan_short<false><<<sg, dim3(256), 0, s>>>(ballots, n, L, m, rounds, meta, ctx->err));
        } else {
            const int32_t chunk = (int32_t)round_up(ceil_div(n, ctx->num_cus), 16);
            const dim3 lg((unsigned)ceil_div(n, chunk));
            if (dtype32)
                SCHULZE_LAUNCH(ctx, K_BALLOT_SCAN, s,
                               k_scan_long<true><<<lg, dim3(1024), 0, s>>>(ballots, n, L, m, chunk, meta, ctx->err));
            else
                SCHULZE_LAUNCH(ctx, K_BALLOT_SCAN, s,
                               k_scan_long<false><<<lg, dim3(1024), 0, s>>>(ballots, n, L, m, chunk, meta, ctx->err));
        }
        if (voter_weight && (rc = weight_total(ctx, s, voter_weight, n, meta.ctr)) != SCHULZE_OK) return rc;
        SCHULZE_LAUNCH(ctx, K_ROUTE, s,
                       k_route<<<dim3(1), dim3(ROUTE_THREADS), 0, s>>>(m, L <= 64 ? L : 0, meta, (int64_t)(trunc_bytes / sizeof(uint32_t)),
                                                             occ_ok ? BUCKETED_PAIR_COST : ATOMIC_PAIR_COST));
        {
            // the m x m accumulator starts at zero unless the device chose the
            // bucketed route and there are no full rankings: then nothing reads it
            const int64_t words = (int64_t)m * m;
            const unsigned fg = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(words / 4 + 1, 256),
                                                                                 (int64_t)ctx->num_cus * 8));
            SCHULZE_LAUNCH(ctx, K_FILL, s,
                           k_fill_acc<<<dim3(fg), dim3(256), 0, s>>>(acc, words, meta, occ_ok && !may_have_full ? 1 : 0));
        }
        if (may_have_full) {
            uint32_t *planes = static_cast<uint32_t *>(ctx->ws[WS_POSITIONS]);
            uint32_t *wplanes = voter_weight ? planes + (size_t)max_groups * full_bits * pitch : nullptr;
            if ((rc = count_dense<true>(ctx, s, ballots, dtype32, n, L, m, pitch, full_bits, max_groups, meta,
                                        voter_weight, planes, wplanes, acc, lda, rsum)) != SCHULZE_OK)
                return rc;
        }
        if (trunc_bytes) {
            uint32_t *planes = static_cast<uint32_t *>(ctx->ws[WS_TRUNC_POS]);
            if ((rc = count_dense<false>(ctx, s, ballots, dtype32, n, L, m, (int32_t)upitch_max, 0, max_groups, meta,
                                         nullptr, planes, nullptr, acc, lda, rsum)) != SCHULZE_OK)
                return rc;
        }
        if (occ_ok) {
            // bucketed pair counting (runs only if the device chose pair scattering)
            char *ob = static_cast<char *>(ctx->ws[WS_OCC]);
            int32_t tbits = 0;
            while ((1 << tbits) < L) ++tbits;
            OccArgs oa{ballots, dtype32, L, m, n, tbits, voter_weight, meta,
                       reinterpret_cast<uint32_t *>(ob + ol.hist),
                       reinterpret_cast<uint32_t *>(ob + ol.row_start),
                       reinterpret_cast<uint4 *>(ob + ol.items),
                       reinterpret_cast<uint32_t *>(ob + ol.item_start),
                       reinterpret_cast<uint32_t *>(ob + ol.tickets), ol.chunk,
                       reinterpret_cast<uint32_t *>(ob + ol.part_start),
                       reinterpret_cast<int32_t *>(ob + ol.fin),
                       reinterpret_cast<uint32_t *>(ob + ol.occ),
                       static_cast<void *>(ob + ol.partial), ol.ppitch,
                       acc, lda, rsum, ctx->err};
            const dim3 g(occ_grid);
            over_flag = reinterpret_cast<uint8_t *>(mb + lay.over);
            if ((rc = occ_bucket<false>(ctx, s, oa, g)) != SCHULZE_OK) return rc;
            SCHULZE_LAUNCH(ctx, K_COUNT_SPARSE, s,
                           k_occ_columns<<<dim3((unsigned)ceil_div(m, 64)), dim3(64 * COL_GROUPS), 0, s>>>(
                               oa, (int32_t)occ_grid));
            SCHULZE_LAUNCH(ctx, K_COUNT_SPARSE, s, k_occ_scan<<<dim3(1), dim3(1024), 0, s>>>(oa));
            const dim3 ig((unsigned)acc_grid);
            if ((rc = occ_bucket<true>(ctx, s, oa, g)) != SCHULZE_OK) return rc;
            if (d_dtype == SCHULZE_U16) {
                if ((rc = occ_accumulate<uint16_t>(ctx, s, oa, ig, m, voter_weight != nullptr, (uint16_t *)d, ldd,
                                                   65535u, over_flag, !may_have_full)) != SCHULZE_OK)
                    return rc;
            } else {
                if ((rc = occ_accumulate<int32_t>(ctx, s, oa, ig, m, voter_weight != nullptr, (int32_t *)d, ldd,
                                                  (uint32_t)INT32_MAX, over_flag, !may_have_full)) != SCHULZE_OK)
                    return rc;
            }
        } else {
            const dim3 pg((unsigned)ceil_div(n, 4));
            if (dtype32)
                SCHULZE_LAUNCH(ctx, K_COUNT_SPARSE, s,
                               k_count_pairs<true><<<pg, dim3(256), 0, s>>>(ballots, L, m, voter_weight, meta, acc, lda,
                                                                            rsum, ctx->err));
            else
                SCHULZE_LAUNCH(ctx, K_COUNT_SPARSE, s,
                               k_count_pairs<false><<<pg, dim3(256), 0, s>>>(ballots, L, m, voter_weight, meta, acc,
                                                                             lda, rsum, ctx->err));
        }
    }
    // rows of the bucketed route were written by it (over_flag given)
    dim3 fgrid((unsigned)m);
    if (d_dtype == SCHULZE_U16) {
        SCHULZE_LAUNCH(ctx, K_COUNT_FINISH, s,
                       k_count_finish<uint16_t><<<fgrid, dim3(256), 0, s>>>(acc, lda, rsum, meta, m, (uint16_t *)d, ldd,
                                                                            65535u, ctx->err, over_flag != nullptr));
    } else {
        SCHULZE_LAUNCH(ctx, K_COUNT_FINISH, s,
                       k_count_finish<int32_t><<<fgrid, dim3(256), 0, s>>>(acc, lda, rsum, meta, m, (int32_t *)d, ldd,
                                                                           (uint32_t)INT32_MAX, ctx->err,
                                                                           over_flag != nullptr));
    }
    return SCHULZE_OK;
}
