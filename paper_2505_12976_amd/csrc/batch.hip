// Batched elections in one persistent launch.
//
// Every election of a batch is one Schulze instance (Section 2.1): its own
// profile, counts d, widest-path closure p, winners and ranking.  A host
// plan turns the batch into a queue of work items; the workgroups of one
// persistent kernel take items in queue order from an atomic ticket:
//
//   scan    ballots of one range of voters -> bit planes of the ranks (32
//           voters per 32-bit word), checked for ids out of range, repeated
//           ids and ids after padding;
//   count   one run of up to 256 sub-blocks of 8 x 8 candidates of one
//           election over one range of voters: per pair (x, y) the mask of
//           the voters with rank(x) < rank(y), one v_bitop3_b32 per bit of
//           the ranks, and its population count.  Complete rankings have no
//           ties, so only sub-blocks with x-block <= y-block are counted and
//           d[y][x] = voters - d[x][y]; elections with truncated ballots
//           count every ordered sub-block;
//   finish  edge weights, closure, beaten-by counts, winners and ranking of
//           one election in one workgroup, started by the workgroup that
//           completes the election's last count item.
//
// The scans of an election come before its counts in the queue (a few
// elections ahead, so that memory-bound scans overlap VALU-bound counts).  A
// count item waits only for the scans of its own election, whose tickets are
// smaller and are held by workgroups that are already running and never
// wait, so every wait ends however many workgroups are resident.  A bounded
// spin turns anything else into a device error.
//
// The closure of the finish runs on a per-workgroup scratch matrix of 16-bit
// elements (counts of elections with at most 65535 voters: half-precision
// keys, or uint16 where a weight is above KEY_MAX) or int32, padded with zero
// rows and columns, by one of two schedules chosen per election size:
// REGISTERS, the plain recurrence with the whole padded matrix (up to
// 192 x 192 uint16 or 128 x 128 int32) held in registers, or TILED(B), the
// three-phase blocked recurrence with B x B tiles run by one workgroup
// (B = 32 and 128 for uint16 only).
#include <algorithm>
#include <new>
#include <numeric>
#include <vector>

#include "fw_tiles.h"
#include "planes.h"

namespace {

using namespace fw;

constexpr int BT = 256;                          // threads per workgroup
constexpr int STAGE_WORDS = 16384;               // count staging: two buffers of rows x cols words
constexpr int SMEM_WORDS = STAGE_WORDS + 1024 + 64;
constexpr int RANGE_PAIRS = 32767;         // voter pairs per count range unless the caller asks for fewer
constexpr int64_t SCAN_WORDS = 1 << 18;    // words (two voters' ranks of a candidate) per scan item
constexpr int SCAN_GROUP_WORDS = 16384;    // words staged at once by a scan
constexpr int SCAN_VEC = 16;              // 16-byte ballot loads in flight per thread
constexpr int SCAN_GROUP_PAIRS = 32;      // voter pairs staged at once by a scan, at most
constexpr int CHUNK_QUADS = 32;            // staged rows of 64 16-byte quads per count chunk
constexpr int64_t SPIN_LIMIT = (int64_t)1 << 24;

enum ItemKind : int32_t { IT_SCAN = 0, IT_COUNT = 1, IT_FINISH = 2 };
enum ElecFlags : int32_t { EF_SQUARE = 1, EF_MULTI = 2, EF_VAL16 = 4, EF_ZERO_D = 8 };

// Per-election parameters (host plan -> device).
struct BElec {
    int64_t ballot_off;  // elements
    int64_t n;           // voters
    int64_t mat_off;     // elements of d and p
    int64_t vec_off;     // elements of is_winner, beaten_by, order
    int64_t pos_off;     // rank-plane words
    int32_t m, L;
    int32_t pitch;        // words per plane row (= 8 * nb8)
    int32_t flags;        // ElecFlags
    int32_t n_scan;       // scan items
    int32_t n_count;      // count items
    int32_t variant;      // closure schedule
    int32_t mp;           // padded closure size
    int32_t nb8;          // blocks of 8 candidates
    int32_t rows;         // plane rows per staged chunk
    int32_t ng;           // column groups of 64 quads in a staged row (1, 2 or 4)
    int32_t vs;           // voter split of small elections (1, 2 or 4)
    int32_t bits;         // planes per group of voters
    int32_t group_pairs;  // voter pairs per group (16, or fewer if the caller asks for smaller ranges)
    int32_t range_groups; // groups per count range
    int32_t scan_pairs;   // voter pairs per scan item (a multiple of group_pairs)
};
static_assert(sizeof(BElec) == 104, "BElec layout");

struct BItem {
    int32_t kind, e, a, b;  // scan: a = first voter pair, b = pairs; count: a = run, b = range
};

// The items are dealt to QUEUES queues by election.  Workgroups are
// dispatched to the dies in turn, so a workgroup starts with the queue of its
// number mod QUEUES: the count items of an election, which read the same
// planes at about the same time, then run on one die and find each other's
// rows in its L2.  A workgroup that finds its queue empty goes on with the next.
constexpr int QUEUES = 8;
constexpr int CTR_STRIDE = 32;                     // one ticket per 128-byte line
constexpr int CTR_ABORT = QUEUES * CTR_STRIDE;     // then the abort word,
constexpr int CTR_ELEC = CTR_ABORT + CTR_STRIDE;   // E scans done and E counts done

struct BatchArgs {
    const BElec *elec;
    const BItem *items;
    int32_t n_items;
    int32_t n_elec;
    int32_t queue[QUEUES + 1];  // first item of each queue
    const void *ballots;
    int32_t dtype32;
    int32_t mode;
    int32_t closure_only;
    uint32_t *planes;
    int32_t *d;
    int32_t *p;
    uint8_t *is_winner;
    int32_t *n_winners;
    int32_t *beaten_by;
    int32_t *order;
    int32_t *level;  // NULL or top-k levels (-1 = not reached)
    int32_t topk;    // rank at least this many candidates per election (0: no levels)
    int32_t pad1;
    int32_t *ctr;  // tickets, abort word, scans and counts done (CTR_*)
    char *scratch;
    int64_t scratch_bytes;  // per workgroup
    int32_t *err;
};

// Every device-memory access of this file goes through FW_GLOBAL pointers, so
// that it compiles to global_* instructions: flat ones would also count as
// LDS operations and every LDS wait would then wait for them too.
template <typename T>
__device__ __forceinline__ FW_GLOBAL T *gmem(T *p) {
    return (FW_GLOBAL T *)p;
}

// LDS of the persistent kernel, used by every function below.  Static (not
// dynamic) so that its address is a constant in every function; a dynamic
// array is located through a table lookup in functions that are not kernels.
__shared__ __attribute__((aligned(16))) uint32_t batch_smem[SMEM_WORDS];

// Candidate id of a ballot entry, -1 for padding.
__device__ inline int32_t ballot_id(int32_t v) { return v < 0 ? -1 : v; }
__device__ inline int32_t ballot_id(uint16_t v) { return v == 0xFFFF ? -1 : (int32_t)v; }

// floor(x / d) for 0 <= x < 2^16 and 1 <= d <= 2^16, with inv = ceil(2^32 / d):
// the error x * (inv - 2^32/d) / 2^32 < 2^-16 <= 1/d never crosses an integer.
__device__ inline uint32_t div_small(uint32_t x, uint32_t inv) { return __umulhi(x, inv); }

// Voter pairs staged at once: whole groups (pitch <= 1024: at least 16 pairs fit)
__host__ __device__ inline int32_t scan_group_pairs(int32_t pitch, int32_t group_pairs) {
    const int32_t fit = SCAN_GROUP_WORDS / pitch < SCAN_GROUP_PAIRS ? SCAN_GROUP_WORDS / pitch : SCAN_GROUP_PAIRS;
    return fit / group_pairs * group_pairs;
}

__device__ inline void abort_all(const BatchArgs &a) {
    __hip_atomic_store(gmem(a.ctr) + CTR_ABORT, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    set_device_error(a.err, SCHULZE_EDEVICE);
}

// ------------------------------------------------------------------ scan
// Voter pairs [q0, q0 + nq) of one election, SCAN_GROUP_WORDS words at a time:
// ranks are scattered into LDS (two voters per word, a row per pair) and each
// column of a group of voters is transposed into its bit planes (planes.h).
// A ballot lists k = (index of its first padding entry) candidates; it is
// valid iff no id follows a padding entry, every listed id is < m, and no id
// is listed twice (the ballots of the item then set as many columns as they
// have entries, which no ballot can exceed).  Complete elections (L >= m - 1)
// also need k >= m - 1: their unset candidate (all ones) is last.
template <typename Id>
__device__ __attribute__((noinline)) void scan_item(const BatchArgs &a, const BElec &el_in, int64_t q0, int64_t nq) {
    // Local copies: a re-read through the references would be a flat load,
    // and every flat load waits for all outstanding global loads.
    const BElec el = el_in;
    uint32_t *smem = batch_smem;
    const FW_GLOBAL Id *ballots = gmem(static_cast<const Id *>(a.ballots));
    const int tid = threadIdx.x;
    const int32_t m = el.m, L = el.L, pitch = el.pitch;
    const bool complete = (el.flags & EF_SQUARE) == 0;
    const int32_t gp = el.group_pairs, bits = el.bits;
    const int32_t vpb = scan_group_pairs(pitch, gp);  // voter pairs staged at once, at most SCAN_GROUP_PAIRS
    uint16_t *buf = reinterpret_cast<uint16_t *>(smem);
    int32_t *first_pad = reinterpret_cast<int32_t *>(smem + SCAN_GROUP_WORDS);  // [2 vpb]
    int32_t *npads = first_pad + 64;
    int32_t *repeated = npads + 64;  // entries less columns set
    const uint32_t inv_l = L > 1 ? (uint32_t)((0x100000000ull + (uint64_t)L - 1) / (uint64_t)L) : 0u;
    const uint32_t inv_p = (uint32_t)((0x100000000ull + (uint64_t)pitch - 1) / (uint64_t)pitch);
    FW_GLOBAL uint32_t *planes = gmem(a.planes + el.pos_off);
    int32_t extra = 0;  // entries less columns set, of this thread
    if (tid == 0) *repeated = 0;

    if ((el.flags & EF_MULTI) && q0 == 0) {  // counts accumulate with atomics: start at zero
        FW_GLOBAL int32_t *D = gmem(a.d + el.mat_off);
        for (int64_t i = tid; i < (int64_t)m * m; i += BT) D[i] = 0;
    }
    bool bad = false;
    // One stage: pairs g .. of the item, its entries and the aligned 16-byte
    // span that covers them (the span's head lies inside the ballot array
    // before them and is skipped).
    constexpr int V = 16 / (int)sizeof(Id);
    struct Stage {
        int32_t npg, nballots, entries, nvec;
        int64_t base, a0;
    };
    auto stage_at = [&](int64_t g) {
        Stage t;
        t.npg = (int32_t)min((int64_t)vpb, q0 + nq - g);
        t.nballots = (int32_t)min((int64_t)2 * t.npg, el.n - 2 * g);
        t.base = el.ballot_off + 2 * g * (int64_t)L;  // ballots of the stage are contiguous
        t.entries = t.nballots * L;                   // < 2^16
        t.a0 = t.base & ~(int64_t)(V - 1);
        const int64_t vend = (t.base + t.entries) & ~(int64_t)(V - 1);
        t.nvec = vend > t.a0 ? (int32_t)((vend - t.a0) / V) : 0;
        return t;
    };
    // SCAN_VEC vectors per thread from vector k0 on, unconditional (clamped),
    // so that all are in flight together
    v4u32 raw[SCAN_VEC];
    auto load = [&](const Stage &t, int32_t k0) {
        const FW_GLOBAL v4u32 *bv = (const FW_GLOBAL v4u32 *)(ballots + t.a0);
        if (t.nvec == 0) return;
#pragma unroll
        for (int j = 0; j < SCAN_VEC; ++j) raw[j] = bv[min(k0 + tid + BT * j, t.nvec - 1)];
    };
    // every rank unset; the transposition leaves it so for the next stage
    for (int32_t w4 = tid; w4 < vpb * pitch / 4; w4 += BT)
        reinterpret_cast<v4u32 *>(smem)[w4] = v4u32{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
    if (tid < 64) {
        first_pad[tid] = L;
        npads[tid] = 0;
    }
    Stage t = stage_at(q0);
    load(t, 0);
    __syncthreads();
    for (int64_t g = q0; g < q0 + nq; g += vpb) {
        const int32_t nballots = t.nballots, entries = t.entries, npg = t.npg;
        const int32_t ngroups = (npg + gp - 1) / gp;
        const int64_t base = t.base, a0 = t.a0;
        extra += tid == 0 ? entries : 0;
        // entry f of the stage: id -> LDS (ballot b = f / L at position t)
        auto take = [&](int32_t f, int32_t id) {
            const int32_t b = (int32_t)div_small((uint32_t)f, inv_l) + (L == 1 ? f : 0);  // inv_l = 0 if L = 1
            const int32_t t = f - b * L;
            if ((uint32_t)id < (uint32_t)m) {
                buf[(b >> 1) * 2 * pitch + 2 * id + (b & 1)] = (uint16_t)t;
                return;
            }
            --extra;
            bad |= id >= m;
            if (id < 0) {  // padding: rare, and never in complete elections' valid ballots
                atomicAdd(&npads[b], 1);
                atomicMin(&first_pad[b], t);
            }
        };
        // Whole vectors of valid ids go straight to LDS; the few others (the
        // span's ends, padding, ids out of range) are read again one by one
        // afterwards, by one copy of the code that handles them: with a copy
        // at every entry the unrolled loop was larger than the instruction
        // cache and took twice as long.
        for (int32_t k0 = 0; k0 < t.nvec; k0 += BT * SCAN_VEC) {
            if (k0) load(t, k0);
            uint32_t rest = 0u;  // vectors left over
#pragma unroll
            for (int j = 0; j < SCAN_VEC; ++j) {
                const int32_t k = k0 + tid + BT * j;
                if (k0 + BT * j >= t.nvec) break;  // (uniform)
                const uint32_t w[4] = {raw[j].x, raw[j].y, raw[j].z, raw[j].w};
                uint32_t top;  // largest id, padding above all
                if constexpr (sizeof(Id) == 2) {
                    const us2 h = __builtin_elementwise_max(
                        __builtin_elementwise_max(__builtin_bit_cast(us2, w[0]), __builtin_bit_cast(us2, w[1])),
                        __builtin_elementwise_max(__builtin_bit_cast(us2, w[2]), __builtin_bit_cast(us2, w[3])));
                    top = max((uint32_t)h.x, (uint32_t)h.y);
                } else {
                    top = max(max(w[0], w[1]), max(w[2], w[3]));
                }
                const int32_t f0 = (int32_t)(a0 + (int64_t)k * V - base);  // entry of the first id (may be < 0)
                if (k >= t.nvec) continue;
                if (f0 < 0 || f0 + V > entries || top >= (uint32_t)m) {
                    rest |= 1u << j;
                    continue;
                }
                // ballot and position of the first id, then stepped
                int32_t b = (int32_t)div_small((uint32_t)f0, inv_l) + (L == 1 ? f0 : 0);
                int32_t pos = f0 - b * L;
                int32_t row = (b >> 1) * 2 * pitch + (b & 1);
                auto id_of = [&](int u) -> uint32_t {
                    if constexpr (sizeof(Id) == 2)
                        return (u & 1) ? w[u >> 1] >> 16 : w[u >> 1] & 0xFFFFu;
                    else
                        return w[u];
                };
                if (pos + V <= L) {
#pragma unroll
                    for (int u = 0; u < V; ++u) buf[row + 2 * id_of(u)] = (uint16_t)(pos + u);
                } else {
#pragma unroll
                    for (int u = 0; u < V; ++u) {
                        buf[row + 2 * id_of(u)] = (uint16_t)pos;
                        if (++pos == L) {
                            pos = 0;
                            ++b;
                            row = (b >> 1) * 2 * pitch + (b & 1);
                        }
                    }
                }
            }
            while (rest) {
                const int j = __builtin_ctz(rest);
                rest &= rest - 1;
                const int64_t at = a0 + (int64_t)(k0 + tid + BT * j) * V;
#pragma unroll 1
                for (int u = 0; u < V; ++u) {
                    const int32_t f = (int32_t)(at + u - base);
                    if (f >= 0 && f < entries) take(f, ballot_id(ballots[at + u]));
                }
            }
        }
        // entries after the last whole vector
        {
            const int64_t vend = a0 + (int64_t)t.nvec * V;
            const int64_t t0 = vend > base ? vend : base;
            const int32_t nt = (int32_t)(base + entries - t0);
            if (tid < nt) take((int32_t)(t0 + tid - base), ballot_id(ballots[t0 + tid]));
        }
        // the next stage's vectors stream in during the transposition
        if (g + vpb < q0 + nq) {
            t = stage_at(g + vpb);
            load(t, 0);
        }
        __syncthreads();
        // a column of a group per thread and step: its pairs' words transposed
        for (int32_t f = tid; f < ngroups * pitch; f += BT) {
            const int32_t j = (int32_t)div_small((uint32_t)f, inv_p), c = f - j * pitch;
            const uint32_t voters = voter_bits(min(2 * gp, nballots - 2 * gp * j));
            uint32_t w[16];
            uint32_t *col = smem + j * gp * pitch + c;
            if (gp == 16) {  // (rows past the last pair are inside the stage; their voters are cleared)
#pragma unroll
                for (int p = 0; p < 16; ++p) w[p] = col[p * pitch];
#pragma unroll
                for (int p = 0; p < 16; ++p) col[p * pitch] = 0xFFFFFFFFu;
            } else {
                for (int p = 0; p < 16; ++p) w[p] = col[min(p, npg - 1 - j * gp) * pitch];
                for (int p = 0; p < gp && j * gp + p < npg; ++p) col[p * pitch] = 0xFFFFFFFFu;
            }
            transpose16(w);
            // ranks are below 1024: the highest bit is that of the columns not set
            if (c < m) extra -= __popc(voters & ~w[15]);
            FW_GLOBAL uint32_t *out = planes + ((g / gp + j) * bits) * (int64_t)pitch + c;
#pragma unroll
            for (int b = 0; b < 10; ++b)
                if (b < bits) out[b * pitch] = w[b] & voters;
        }
        if (tid < nballots) {
            const int32_t k = first_pad[tid];
            if (L - npads[tid] != k || (complete && k < m - 1)) bad = true;
            first_pad[tid] = L;
            npads[tid] = 0;
        }
        __syncthreads();
    }
    for (int off = 32; off >= 1; off >>= 1) extra += __shfl_xor(extra, off);
    if ((tid & 63) == 0 && extra) atomicAdd(repeated, extra);
    __syncthreads();
    if (tid == 0 && *repeated != 0) bad = true;
    if (bad) set_device_error(a.err, SCHULZE_EBALLOT);
}

// ------------------------------------------------------------------ count
__device__ inline void sub_coords(int32_t s, int32_t nb8, bool square, int32_t &bx, int32_t &by) {
    if (square) {
        bx = s / nb8;
        by = s - bx * nb8;
        return;
    }
    int32_t x = 0, start = 0;
    while (start + (nb8 - x) <= s) {
        start += nb8 - x;
        ++x;
    }
    bx = x;
    by = x + (s - start);
}

__device__ void finish(const BatchArgs &a, const BElec &el, int32_t e);

// Sub-blocks [run * per_phase, ...) of election e over the groups of voters of
// range `range`, on bit planes: a thread's 8 x 8 sub-block takes 64
// v_bitop3_b32 per plane row for the masks of the voters that prefer x to y
// and 64 population counts per group (the single-election count has the
// rates).  Staged rows hold columns c0 .. 8 nb8 - 1 of consecutive plane rows,
// streamed into LDS without passing through registers, each 8-column block
// split into two 16-byte halves stored in separate row halves so that
// neighbouring sub-blocks read neighbouring 16 bytes.
__device__ __attribute__((noinline)) void count_item(const BatchArgs &a, const BElec &el_in, int32_t e, int32_t run,
                                                    int32_t range) {
    const BElec el = el_in;  // local copy (see scan_item)
    const int64_t pitch = el.pitch;
    uint32_t *smem = batch_smem;
    __shared__ int32_t sh_flag;
    const int tid = threadIdx.x;
    const bool square = (el.flags & EF_SQUARE) != 0;
    const bool multi = (el.flags & EF_MULTI) != 0;
    const int32_t m = el.m, nb8 = el.nb8;
    const int32_t vs = el.vs, per_phase = BT / vs;
    const int32_t phase = tid / per_phase, sub = tid - phase * per_phase;
    const int32_t S = square ? nb8 * nb8 : nb8 * (nb8 + 1) / 2;
    const int32_t s_first = run * per_phase;
    const int32_t s_mine = s_first + sub;
    const bool active = s_mine < S;
    int32_t bx0, by0;
    sub_coords(s_first, nb8, square, bx0, by0);
    const int32_t cb0 = square ? 0 : bx0;  // first staged block of 8 columns
    int32_t bx = cb0, by = cb0;
    if (active) sub_coords(s_mine, nb8, square, bx, by);
    const int32_t c0 = 8 * cb0;
    const int32_t cols = 8 * (nb8 - cb0);
    const int32_t half = cols / 2;
    const int32_t nq = cols / 4;  // 16-byte quads per staged row
    const int32_t bits = el.bits, ROWS = el.rows;  // ROWS * cols <= STAGE_WORDS / 2
    const int64_t gv = 2 * el.group_pairs;         // voters per group
    const int64_t g0 = (int64_t)range * el.range_groups;
    const int64_t g1 = min((el.n + gv - 1) / gv, g0 + el.range_groups);
    const uint32_t nv = (uint32_t)(min(el.n, gv * g1) - gv * g0);
    const int32_t nrows = (int32_t)(g1 - g0) * bits;  // (at most RANGE_PAIRS / group_pairs groups of at most 10 planes)
    const FW_GLOBAL uint32_t *src = gmem(a.planes + el.pos_off) + g0 * bits * pitch + c0;
    uint32_t *stage = smem;

    // the scans of this election must be complete
    if (tid == 0) {
        int32_t ok = 1;
        int64_t spins = 0;
        FW_GLOBAL int32_t *ctr = gmem(a.ctr);
        while (__hip_atomic_load(ctr + CTR_ELEC + e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < el.n_scan) {
            if (__hip_atomic_load(ctr + CTR_ABORT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 || ++spins > SPIN_LIMIT) {
                abort_all(a);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        sh_flag = ok;
    }
    __syncthreads();
    if (!sh_flag) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");

    uint32_t acc[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = 0u;
    Masks lt;
    lt.clear();

    // rows r0 .. of the range to LDS buffer st: a wavefront takes every
    // fourth row, 64 quads per instruction; LDS quad i of a row is its
    // global quad 2 i (first halves) or 2 (i - nq / 2) + 1
    FW_LDS uint32_t *const lds = (FW_LDS uint32_t *)stage;
    const int32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto fill = [&](int32_t r0, FW_LDS uint32_t *st) {
        int ti = tid;
        asm volatile("" : "+v"(ti));  // (addresses built here, not kept in registers)
        const int32_t lane = ti & 63, rend = min(ROWS, nrows - r0);
        for (int32_t r = wave; r < rend; r += 4) {
            const FW_GLOBAL uint32_t *row = src + (int64_t)(r0 + r) * pitch;
            for (int32_t q = 0; q < nq; q += 64) {
                const int32_t i = q + lane;
                if (i < nq)
                    __builtin_amdgcn_global_load_lds(row + 4 * (i < nq / 2 ? 2 * i : 2 * (i - nq / 2) + 1),
                                                     st + r * cols + 4 * q, 16, 0, 0);
            }
        }
    };
    struct Row {
        v4u32 x[2], y[2];
    };
    auto read = [&](const FW_LDS uint32_t *xp, const FW_LDS uint32_t *yp, Row &q) {
        q.x[0] = *(const FW_LDS v4u32 *)xp;
        q.x[1] = *(const FW_LDS v4u32 *)(xp + half);
        q.y[0] = *(const FW_LDS v4u32 *)yp;
        q.y[1] = *(const FW_LDS v4u32 *)(yp + half);
    };

    // Two stage buffers: one chunk is counted while the next streams in, one
    // barrier per chunk.  With the voters split (vs > 1) a chunk holds whole
    // groups and each phase takes every vs-th of them; otherwise a group may
    // go on in the next chunk.
    const int32_t xo = (bx - cb0) * 4, yo = (by - cb0) * 4;
    __syncthreads();  // the stage is free (a previous item of this workgroup may have used it)
    fill(0, lds);
    int32_t cur = 0, b = 0;  // b: planes of the current group done
    for (int32_t r0 = 0; r0 < nrows; r0 += ROWS) {
        __builtin_amdgcn_s_waitcnt(0);  // this wavefront's pieces of the chunk are in LDS
        __syncthreads();                // everyone's are, and the chunk before is consumed
        FW_LDS uint32_t *st = lds + cur * (STAGE_WORDS / 2);
        cur ^= 1;
        if (r0 + ROWS < nrows) fill(r0 + ROWS, lds + cur * (STAGE_WORDS / 2));
        const int32_t rend = min(ROWS, nrows - r0);
        if (!active) continue;
        for (int32_t r = phase * bits; r < rend;) {
            const int32_t take = min(bits - b, rend - r);
            const FW_LDS uint32_t *xp = st + r * cols + xo, *yp = st + r * cols + yo;
            Row q0, q1;
            read(xp, yp, q0);
#pragma unroll 1
            for (int32_t k = 0; k + 1 < take; k += 2) {
                read(xp + cols, yp + cols, q1);
                __builtin_amdgcn_sched_barrier(0);
                lt.step(q0.x, q0.y);
                __builtin_amdgcn_sched_barrier(0);
                const int32_t on = k + 2 < take ? 2 * cols : 0;  // (after the last row: a row again, unused)
                xp += on;
                yp += on;
                read(xp, yp, q0);
                __builtin_amdgcn_sched_barrier(0);
                lt.step(q1.x, q1.y);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (take & 1) lt.step(q0.x, q0.y);
            r += take;
            b += take;
            if (b == bits) {
                lt.count(acc);
                lt.clear();
                b = 0;
                r += (vs - 1) * bits;
            }
        }
    }
    __syncthreads();  // the stage is consumed: the phases' counts go there
    if (vs > 1 && phase > 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) stage[((phase - 1) * 64 + i * 8 + j) * per_phase + sub] = acc[i][j];
    }
    __syncthreads();
    if (phase == 0 && active) {
        if (vs > 1) {
            for (int32_t ph = 1; ph < vs; ++ph)
#pragma unroll
                for (int i = 0; i < 8; ++i)
#pragma unroll
                    for (int j = 0; j < 8; ++j) acc[i][j] += stage[((ph - 1) * 64 + i * 8 + j) * per_phase + sub];
        }
        FW_GLOBAL int32_t *D = gmem(a.d + el.mat_off);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int32_t x = 8 * bx + i;
            if (x >= m) continue;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int32_t y = 8 * by + j;
                if (y >= m) continue;
                const uint32_t cnt = acc[i][j];
                if (square) {
                    if (x == y) {
                        if (!multi) D[(int64_t)x * m + y] = 0;
                    } else if (multi) {
                        __hip_atomic_fetch_add(D + (int64_t)x * m + y, (int32_t)cnt, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                    } else {
                        D[(int64_t)x * m + y] = (int32_t)cnt;
                    }
                } else if (x < y) {
                    if (multi) {
                        __hip_atomic_fetch_add(D + (int64_t)x * m + y, (int32_t)cnt, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                        __hip_atomic_fetch_add(D + (int64_t)y * m + x, (int32_t)(nv - cnt), __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                    } else {
                        D[(int64_t)x * m + y] = (int32_t)cnt;
                        D[(int64_t)y * m + x] = (int32_t)(nv - cnt);
                    }
                } else if (x == y && !multi) {
                    D[(int64_t)x * m + x] = 0;
                }
            }
        }
    }

    // completion: the workgroup that finishes the election's last count item
    // runs its finish.  An election of one count item needs nothing from
    // other workgroups: the release writes back every dirty line of the die's
    // L2, about a microsecond that its workgroups take in turn (4096 elections
    // of at most 10 candidates: 1249 us with it).
    if (el.n_count > 1) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __syncthreads();
        if (tid == 0)
            sh_flag = __hip_atomic_fetch_add(gmem(a.ctr) + CTR_ELEC + a.n_elec + e, 1, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT) == el.n_count - 1;
        __syncthreads();
        if (!sh_flag) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    } else {
        __syncthreads();
    }
    finish(a, el, e);
}

// ------------------------------------------------------------------ finish
// Blocked recurrence of one workgroup over an mp x mp matrix (mp a multiple
// of B): per round r the diagonal tile is closed, then the panels of block
// row and column r, then the rest; every tile becomes
// max(P[I][J], P[I][r] (x) P[r][J]).
template <typename E, int B>
__device__ __attribute__((noinline)) void closure_tiled(E *P_, int32_t mp) {
    FW_GLOBAL E *P = gmem(P_);
    E *lds = reinterpret_cast<E *>(batch_smem);
    const int32_t nb = mp / B;
    auto tile = [&](int32_t I, int32_t J) { return P + (int64_t)I * B * mp + (int64_t)J * B; };
    for (int32_t r = 0; r < nb; ++r) {
        diag_close<E, B>(tile(r, r), mp, tile(r, r), mp, nullptr, 0, lds);
        for (int32_t t = 0; t < 2 * (nb - 1); ++t) {
            int32_t I, J;
            if (t < nb - 1) {
                I = r;
                J = t < r ? t : t + 1;
            } else {
                const int32_t u = t - (nb - 1);
                J = r;
                I = u < r ? u : u + 1;
            }
            Acc<E, B> acc;
            acc_load<E, B>(acc, tile(I, J), mp);
            acc_product<E, B>(acc, tile(I, r), mp, tile(r, J), mp, lds);
            acc_store<E, B>(acc, tile(I, J), mp);
        }
        for (int32_t t = 0; t < (nb - 1) * (nb - 1); ++t) {
            const int32_t i = t / (nb - 1), j = t % (nb - 1);
            const int32_t I = i < r ? i : i + 1, J = j < r ? j : j + 1;
            Acc<E, B> acc;
            acc_load<E, B>(acc, tile(I, J), mp);
            acc_product<E, B>(acc, tile(I, r), mp, tile(r, J), mp, lds);
            acc_store<E, B>(acc, tile(I, J), mp);
        }
        __syncthreads();
    }
}

// The same recurrence for 16-bit elements and B = 64 with the operand tiles
// streamed into LDS while the product before them runs (two slots each of A
// and B, refilled only when the next product needs another tile; the next
// output tile's elements come into registers).  One workgroup closes the
// whole matrix and only one other shares its CU, so nothing else hides the
// waits.  One election of m = 448 in every workgroup, uint16 and each
// product's tiles copied through registers first: 2500 us; half-precision
// keys and streamed: 1730 (the 205 MB of the matrices, re-read and rewritten
// each round, at 2.9 TB/s); top-3 of 167 elections of m <= 410: 6550 and
// 4810 us.
// A's rows are 128 bytes; the 16-byte pieces of row R sit at piece ^ 2 ((R / 4)
// % 4), so that the four rows that a wavefront reads together fall on
// different banks.
template <typename E>
struct Stream64 {
    using L = Lane<E>;
    using W = typename L::W;
    static constexpr int TILE = 64 * 64;
    static constexpr int LDS_ELEMS = 4 * TILE;

    // this thread's element offsets in a tile of pitch mp <= SCHULZE_BATCH_MAX_M
    // (so that no product of the pitch is left in the loops)
    struct Offsets {
        uint32_t a, b;  // first operand piece (A swizzled), + 32 mp: the second
        uint32_t c;     // first of four output rows
    };
    __device__ static Offsets offsets(int32_t mp) {
        const uint32_t t = threadIdx.x, l = t & 63, row = 8 * (t >> 6) + (l >> 3);
        const uint32_t tx = t & 15, ty = t >> 4;
        // (row and row + 32 have the same swizzle)
        return Offsets{row * mp + 8 * ((l & 7) ^ (((row >> 2) & 3) << 1)), row * mp + 8 * (l & 7),
                       4 * ty * mp + 4 * tx};
    }
    // 64 x 64 elements at src into lds; a wavefront instruction moves 8 rows
    __device__ static void tile_in(FW_GLOBAL const E *src, uint32_t off, int32_t mp, FW_LDS E *lds) {
        const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        __builtin_amdgcn_global_load_lds(src + off, lds + w * 512, 16, 0, 0);
        __builtin_amdgcn_global_load_lds(src + 32 * mp + off, lds + (w + 4) * 512, 16, 0, 0);
    }
    // the thread's 4 x 4 output elements: one 8-byte access a row
    __device__ static void out_load(Acc<E, 64> &c, FW_GLOBAL const E *tile, uint32_t off, int32_t mp) {
        for (int i = 0; i < 4; ++i) {
            const v2u32 x = *retype<const v2u32>(tile + i * mp + off);
            const uint32_t x0 = x.x, x1 = x.y;
            c.c[i][0] = __builtin_bit_cast(W, x0);
            c.c[i][1] = __builtin_bit_cast(W, x1);
        }
    }
    __device__ static void out_store(const Acc<E, 64> &c, FW_GLOBAL E *tile, uint32_t off, int32_t mp) {
        for (int i = 0; i < 4; ++i)
            *retype<v2u32>(tile + i * mp + off) =
                v2u32{__builtin_bit_cast(uint32_t, c.c[i][0]), __builtin_bit_cast(uint32_t, c.c[i][1])};
    }

    using Step = Step64<E>;
    __device__ static void step_in(Step &s, const FW_LDS E *As, const FW_LDS E *Bs, int k, int tx, int ty) {
        const int piece = (k >> 3) ^ ((ty & 3) << 1);
        for (int i = 0; i < 4; ++i) s.a[i] = *(const FW_LDS v2u32 *)(As + (4 * ty + i) * 64 + piece * 8 + (k & 7));
        for (int q = 0; q < 4; ++q) {
            const FW_LDS W *b = (const FW_LDS W *)(Bs + (k + q) * 64 + 4 * tx);
            s.b[q][0] = b[0];
            s.b[q][1] = b[1];
        }
    }
    // c = max(c, A (x) B); the next step's operands are read before this one's products
    __device__ static void product(Acc<E, 64> &c, const FW_LDS E *As, const FW_LDS E *Bs) {
        const int t = lane_tid(), tx = t & 15, ty = t >> 4;
        Step s0, s1;
        step_in(s0, As, Bs, 0, tx, ty);
#pragma unroll 1
        for (int k = 0; k < 64; k += 8) {
            step_in(s1, As, Bs, k + 4, tx, ty);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xC47F);  // lgkmcnt(4): s0 is in (a step is four LDS reads)
            __builtin_amdgcn_sched_barrier(0);
            s0.add(c);
            __builtin_amdgcn_sched_barrier(0);
            step_in(s0, As, Bs, (k + 8) & 63, tx, ty);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0xC47F);
            __builtin_amdgcn_sched_barrier(0);
            s1.add(c);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

template <typename E>
__device__ __attribute__((noinline)) void closure_stream64(E *P_, int32_t mp) {
    using S = Stream64<E>;
    FW_GLOBAL E *P = scalar_ptr(gmem(P_));
    mp = __builtin_amdgcn_readfirstlane(mp);  // (uniform: scalar addresses and loops)
    FW_LDS E *As = (FW_LDS E *)reinterpret_cast<E *>(batch_smem), *Bs = As + 2 * S::TILE;
    const int32_t nb = mp / 64;
    auto tile = [&](int32_t I, int32_t J) { return P + (uint32_t)(64 * (I * mp + J)); };
    const typename S::Offsets off = S::offsets(mp);
    // count output tiles at(t) = (I, J), each with A = (I, r) and B = (r, J);
    // no tile is both an output and the operand of another one
    auto run = [&](int32_t count, int32_t r, auto at) {
        if (count == 0) return;
        int32_t I, J, sa = 0, sb = 0;
        at(0, I, J);
        Acc<E, 64> c, next;
        __syncthreads();  // the tiles are stored and the LDS is free
        S::tile_in(tile(I, r), off.a, mp, As);
        S::tile_in(tile(r, J), off.b, mp, Bs);
        S::out_load(next, tile(I, J), off.c, mp);
        int32_t I0 = I, J0 = J;
#pragma unroll 1
        for (int32_t t = 0; t < count; ++t) {
            __builtin_amdgcn_s_waitcnt(0);  // this wave's pieces of the operands are in LDS
            __syncthreads();                // everyone's are, and the other slots are consumed
            // (the last product is stored here, not before the wait above)
            if (t > 0) S::out_store(c, tile(I0, J0), off.c, mp);
            c = next;
            I0 = I;
            J0 = J;
            const FW_LDS E *A = As + sa * S::TILE, *B = Bs + sb * S::TILE;
            at(min(t + 1, count - 1), I, J);  // (the last one again: nothing to fetch, a load that is not used)
            if (I != I0) S::tile_in(tile(I, r), off.a, mp, As + (sa ^= 1) * S::TILE);
            if (J != J0) S::tile_in(tile(r, J), off.b, mp, Bs + (sb ^= 1) * S::TILE);
            S::out_load(next, tile(I, J), off.c, mp);
            S::product(c, A, B);
        }
        S::out_store(c, tile(I0, J0), off.c, mp);
    };
    for (int32_t r = 0; r < nb; ++r) {
        diag_close<E, 64>(tile(r, r), mp, tile(r, r), mp, nullptr, 0, reinterpret_cast<E *>(batch_smem));
        const int32_t o = nb - 1;
        run(2 * o, r, [&](int32_t t, int32_t &I, int32_t &J) {
            const int32_t u = t < o ? t : t - o, x = u < r ? u : u + 1;
            I = t < o ? r : x;
            J = t < o ? x : r;
        });
        run(o * o, r, [&](int32_t t, int32_t &I, int32_t &J) {
            const int32_t i = t / o, j = t - i * o;
            I = i < r ? i : i + 1;
            J = j < r ? j : j + 1;
        });
        __syncthreads();
    }
}

static_assert((2 * 64 * 65 + 2 * SCHULZE_BATCH_MAX_M) % 4 == 0 &&
                  2 * 64 * 65 + 2 * SCHULZE_BATCH_MAX_M + Diag<int32_t, 64>::LDS_ELEMS <= SMEM_WORDS,
              "LDS of the one-tile finish (its buffer 16-byte aligned)");
static_assert(Stream64<_Float16>::LDS_ELEMS * 2 <= SMEM_WORDS * 4, "streamed closure LDS");
static_assert(2 * CHUNK_QUADS * 64 * 4 <= STAGE_WORDS, "two count stage buffers: rows * cols <= 32 / ng * 256 ng words each");
static_assert(diag_lds_elems<uint16_t, 192>() * 2 <= SMEM_WORDS * 4 && diag_lds_elems<int32_t, 128>() * 4 <= SMEM_WORDS * 4,
              "diagonal closure LDS");

// Each schedule is its own function: inlined together, their register
// demands would be allocated as one and spill.
template <typename E, int B>
__device__ __attribute__((noinline)) void closure_reg(E *P_, int32_t mp) {
    FW_GLOBAL E *P = gmem(P_);
    diag_close<E, B>(P, mp, P, mp, nullptr, 0, reinterpret_cast<E *>(batch_smem));
}

template <typename E>
__device__ void closure_dispatch(E *P, int32_t mp, int32_t variant) {
    if (variant == SCHULZE_BATCH_CLOSURE_REGISTERS) {
        switch (mp) {
            case 32: closure_reg<E, 32>(P, mp); break;
            case 64: closure_reg<E, 64>(P, mp); break;
            case 96: closure_reg<E, 96>(P, mp); break;
            case 128: closure_reg<E, 128>(P, mp); break;
            default:
                if constexpr (sizeof(E) == 2) {
                    switch (mp) {
                        case 160: closure_reg<E, 160>(P, mp); break;
                        case 192: closure_reg<E, 192>(P, mp); break;
                        default: break;
                    }
                }
                break;
        }
    } else if (variant == SCHULZE_BATCH_CLOSURE_TILED32) {
        if constexpr (sizeof(E) == 2) closure_tiled<E, 32>(P, mp);
    } else if (variant == SCHULZE_BATCH_CLOSURE_TILED64) {
        if constexpr (sizeof(E) == 2)
            closure_stream64<E>(P, mp);
        else
            closure_tiled<E, 64>(P, mp);
    } else {
        if constexpr (sizeof(E) == 2) closure_tiled<E, 128>(P, mp);
    }
}

// An entry of the scratch matrix as the integer it stands for (half-precision
// keys: of the values up to KEY_MAX; no branch, so that loads before it stay
// in flight together).
template <typename E>
__device__ __forceinline__ int32_t value_of(E x) {
    if constexpr (__is_same(E, _Float16)) {
        const int32_t k = __builtin_bit_cast(int16_t, x), sign = k >> 15;
        return 31744 + (((k & 0x7FFF) ^ sign) - sign);
    } else {
        return (int32_t)x;
    }
}

// false (half-precision keys only): a weight is above KEY_MAX and nothing
// has been written.  SMALL (16, 32, 48 or 64, int32): the whole matrix is one tile of
// the register closure, so the counts stay in LDS and every level's weights,
// closure and beaten-by counts run on them there, without the scratch matrix
// (200 elections of at most 48 candidates, top-3: 151 -> 129 us).
template <typename E, int SMALL = 0>
__device__ bool finish_t(const BatchArgs &a, const BElec &el, int32_t e, uint32_t *smem) {
    const int tid = threadIdx.x;
    const int32_t m = el.m, mp = el.mp;
    const int32_t mode = a.mode;
    FW_GLOBAL uint8_t *is_winner = gmem(a.is_winner);
    FW_GLOBAL int32_t *beaten_by = a.beaten_by ? gmem(a.beaten_by) : nullptr;
    FW_GLOBAL int32_t *order = a.order ? gmem(a.order) : nullptr;
    FW_GLOBAL int32_t *p_out = a.p ? gmem(a.p) : nullptr;
    E *Pv = reinterpret_cast<E *>(a.scratch + (int64_t)blockIdx.x * a.scratch_bytes);
    FW_GLOBAL E *P = gmem(Pv);
    FW_GLOBAL int32_t *D = gmem(a.d + el.mat_off);
    if ((el.flags & EF_ZERO_D) && !a.closure_only) {  // no voters: d = 0
        for (int64_t i = tid; i < (int64_t)m * m; i += BT) D[i] = 0;
        __syncthreads();
    }

    // edge weights into the padded scratch matrix, 64 x 64 tiles through LDS;
    // candidates with gone[x] >= 0 (removed for top-k) lose all their edges
    int32_t *ta = reinterpret_cast<int32_t *>(smem);  // [64][65]
    int32_t *tb = ta + 64 * 65;                       // [64][65]
    int32_t *bb = tb + 64 * 65;                       // [SCHULZE_BATCH_MAX_M]
    int32_t *lvl = bb + SCHULZE_BATCH_MAX_M;          // [SCHULZE_BATCH_MAX_M]
    const int32_t nt = (mp + 63) / 64;
    // both tiles of a pair (I, J), (J, I) at once: each is read once.  All 32
    // loads are in flight together, with addresses clamped into the matrix (a
    // conditional load would wait for the ones before it); entries outside
    // the m x m matrix are 0
    auto pair_in = [&](int32_t I, int32_t J, auto at) {
        __syncthreads();
        constexpr int PER = 64 * 64 / BT;
        int32_t va[PER], vb[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int q = tid + k * BT, r = q >> 6, c = q & 63;
            va[k] = at(min(I * 64 + r, m - 1), min(J * 64 + c, m - 1));
            vb[k] = at(min(J * 64 + r, m - 1), min(I * 64 + c, m - 1));
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int q = tid + k * BT, r = q >> 6, c = q & 63;
            ta[r * 65 + c] = I * 64 + r < m && J * 64 + c < m ? va[k] : 0;
            tb[r * 65 + c] = J * 64 + r < m && I * 64 + c < m ? vb[k] : 0;
        }
        __syncthreads();
    };
    // false: a weight is above KEY_MAX (half-precision keys)
    auto weights = [&](const int32_t *gone) -> bool {
        bool too_big = false, wide = false;
        auto out = [&](int32_t I, int32_t J, const int32_t *fw, const int32_t *bw) {
            for (int q = tid; q < 64 * 64; q += BT) {
                const int r = q >> 6, c = q & 63;
                const int32_t i = I * 64 + r, j = J * 64 + c;
                if (i >= mp || j >= mp) continue;
                const int32_t x = fw[r * 65 + c], y = bw[c * 65 + r];  // d[i][j], d[j][i]
                int32_t w = 0;
                if (i != j && x > y) w = mode == SCHULZE_MARGIN ? x - y : x;
                if (gone && w && (gone[i] >= 0 || gone[j] >= 0)) w = 0;
                if constexpr (sizeof(E) == 2) {
                    if ((uint32_t)w > 65535u) {  // counts above the bound the plan assumed
                        too_big = true;
                        w = 65535;
                    }
                }
                if constexpr (__is_same(E, _Float16)) {
                    wide = wide || w > (int32_t)KEY_MAX;
                    P[(int64_t)i * mp + j] = __builtin_bit_cast(E, key_of((uint32_t)w));
                } else {
                    P[(int64_t)i * mp + j] = (E)w;
                }
            }
        };
        for (int32_t I = 0; I < nt; ++I) {
            for (int32_t J = I; J < nt; ++J) {
                pair_in(I, J, [&](int32_t i, int32_t j) { return D[(int64_t)i * m + j]; });
                out(I, J, ta, tb);
                if (I != J) out(J, I, tb, ta);
            }
        }
        if constexpr (__is_same(E, _Float16)) {
            if (__syncthreads_or(wide)) return false;
        }
        if (too_big) set_device_error(a.err, SCHULZE_ERANGE);
        __syncthreads();
        return true;
    };
    // bb[x] = #{y : P[y][x] > P[x][y]}
    auto beaten = [&]() {
        for (int32_t x = tid; x < m; x += BT) bb[x] = 0;
        const int32_t mt = (m + 63) / 64;
        for (int32_t I = 0; I < mt; ++I) {
            for (int32_t J = I; J < mt; ++J) {
                pair_in(I, J, [&](int32_t i, int32_t j) { return value_of<E>(P[(int64_t)i * mp + j]); });
                // lane c of wavefront g: candidate y = (J, c) against x = (I, r) for r = g, g + 4, ..
                const int32_t c = tid & 63, g = tid >> 6;
                const int32_t y = J * 64 + c;
                int32_t cnt = 0, other = 0;  // (other: lane q holds the count of x = (I, g + 4 q))
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int32_t r = g + 4 * q;
                    const int32_t pxy = ta[r * 65 + c], pyx = tb[c * 65 + r];
                    cnt += pxy > pyx ? 1 : 0;
                    const int32_t beats = (int32_t)__popcll(__ballot(pyx > pxy));
                    other = c == q ? beats : other;
                }
                // (on a diagonal block the lanes' counts see every pair from both sides)
                if (I != J && c < 16 && other) atomicAdd(&bb[I * 64 + g + 4 * c], other);
                if (y < m && cnt) atomicAdd(&bb[y], cnt);
            }
        }
        __syncthreads();
    };

    // one level: closure of the weights without the candidates gone, and bb
    constexpr int SP = SMALL + 1;  // LDS pitch of the one tile: counts in ta, closure in tb
    auto level = [&](const int32_t *gone) -> bool {
        if constexpr (SMALL > 0) {
            using Dg = Diag<E, SMALL>;
            static_assert(sizeof(E) == 4 && 64 * 65 >= SMALL * SP, "one int32 tile");
            const int tx = tid & 15, ty = tid >> 4;
            FW_LDS E *buf = (FW_LDS E *)(lvl + SCHULZE_BATCH_MAX_M);
            typename Dg::W v[Dg::RA][Dg::WC];
            bool too_big = false;
            for (int r = 0; r < Dg::RA; ++r)
                for (int c = 0; c < Dg::WC; ++c) {
                    const int i = ty + 16 * r, j = tx + 16 * c;
                    const int32_t x = ta[i * SP + j], y = ta[j * SP + i];
                    int32_t w = 0;
                    if (i != j && x > y) w = mode == SCHULZE_MARGIN ? x - y : x;
                    if (gone && w && (gone[i] >= 0 || gone[j] >= 0)) w = 0;
                    if ((el.flags & EF_VAL16) && (uint32_t)w > 65535u) {  // counts above the bound the plan assumed
                        too_big = true;
                        w = 65535;
                    }
                    v[r][c] = w;
                }
            if (too_big) set_device_error(a.err, SCHULZE_ERANGE);
            Dg::template publish<0>(v, 0, buf, tx, ty);
            Dg::template steps<0>(v, tx, ty, buf);
            for (int r = 0; r < Dg::RA; ++r)
                for (int c = 0; c < Dg::WC; ++c) tb[(ty + 16 * r) * SP + tx + 16 * c] = v[r][c];
            for (int32_t x = tid; x < SMALL; x += BT) bb[x] = 0;
            __syncthreads();
            constexpr int PARTS = BT / SMALL;
            const int x = tid % SMALL, part = tid / SMALL;
            int32_t cnt = 0;
            for (int y = part; y < SMALL && part < PARTS; y += PARTS) cnt += tb[y * SP + x] > tb[x * SP + y] ? 1 : 0;
            if (cnt) atomicAdd(&bb[x], cnt);
            __syncthreads();
            return true;
        } else {
            if (!weights(gone)) return false;
            closure_dispatch<E>(Pv, mp, el.variant);
            __syncthreads();
            beaten();
            return true;
        }
    };
    if constexpr (SMALL > 0) {
        constexpr int PER = SMALL * SMALL / BT;
        int32_t v[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int q = tid + k * BT;
            v[k] = D[(int64_t)min(q / SMALL, m - 1) * m + min(q % SMALL, m - 1)];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int q = tid + k * BT, i = q / SMALL, j = q % SMALL;
            ta[i * SP + j] = i < m && j < m ? v[k] : 0;
        }
        __syncthreads();
    }

    if (!level(nullptr)) return false;

    __shared__ int32_t sh_wins;
    if (tid == 0) sh_wins = 0;
    __syncthreads();
    int32_t wins = 0;
    for (int32_t x = tid; x < m; x += BT) {
        const int32_t bx = bb[x];
        const bool win = bx == 0;
        wins += win ? 1 : 0;
        is_winner[el.vec_off + x] = win ? 1 : 0;
        if (beaten_by) beaten_by[el.vec_off + x] = bx;
        if (order) {
            int32_t rank = 0;
            for (int32_t y = 0; y < m; ++y) {
                const int32_t by = bb[y];
                rank += (by < bx || (by == bx && y < x)) ? 1 : 0;
            }
            order[el.vec_off + rank] = x;
        }
    }
    if (wins) atomicAdd(&sh_wins, wins);
    if (p_out) {
        // eight rows at a time, their loads (clamped) before their stores
        FW_GLOBAL int32_t *Pout = p_out + el.mat_off;
        constexpr int R = 8, H = SCHULZE_BATCH_MAX_M / BT;
        for (int32_t x0 = 0; x0 < m; x0 += R) {
            int32_t v[R][H];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int h = 0; h < H; ++h)
                    v[r][h] = SMALL > 0 ? tb[min(x0 + r, m - 1) * SP + min(tid + h * BT, m - 1)]
                                        : value_of<E>(P[(int64_t)min(x0 + r, m - 1) * mp + min(tid + h * BT, m - 1)]);
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const int32_t x = x0 + r, y = tid + h * BT;
                    if (x < m && y < m) Pout[(int64_t)x * m + y] = x == y ? 0 : v[r][h];
                }
        }
    }
    __syncthreads();
    if (tid == 0 && a.n_winners) gmem(a.n_winners)[e] = sh_wins;

    // top-k by iterated winner removal: level 0 = the winners; each further
    // level closes the weights with the ranked candidates' edges deleted and
    // takes the winners among the candidates left
    if (a.level && a.topk > 0) {
        __shared__ int32_t sh_ranked, sh_new;
        for (int32_t x = tid; x < (SMALL > 0 ? SMALL : m); x += BT) lvl[x] = bb[x] == 0 ? 0 : -1;
        if (tid == 0) sh_ranked = sh_wins;
        __syncthreads();
        // every nonempty set of candidates has a winner, so each level ranks at least one
        for (int32_t rank = 1; rank < m && sh_ranked < a.topk && sh_ranked < m; ++rank) {
            level(lvl);  // (some of the first level's weights)
            if (tid == 0) sh_new = 0;
            __syncthreads();
            int32_t got = 0;
            for (int32_t x = tid; x < m; x += BT)
                if (lvl[x] < 0 && bb[x] == 0) {  // removed candidates have no edges: skip them
                    lvl[x] = rank;
                    ++got;
                }
            if (got) atomicAdd(&sh_new, got);
            __syncthreads();
            if (tid == 0) sh_ranked += sh_new;
            __syncthreads();
        }
        FW_GLOBAL int32_t *lv = gmem(a.level);
        for (int32_t x = tid; x < m; x += BT) lv[el.vec_off + x] = lvl[x];
    }
    __syncthreads();
    return true;
}

__device__ __attribute__((noinline)) void finish(const BatchArgs &a, const BElec &el_in, int32_t e) {
    const BElec el = el_in;  // local copy (see scan_item)
    // 16-bit values: half-precision keys, unless a weight is above KEY_MAX; one
    // tile of the register closure: integers in LDS
    if (el.variant == SCHULZE_BATCH_CLOSURE_REGISTERS && el.mp <= 64) {
        if (el.m <= 16)
            finish_t<int32_t, 16>(a, el, e, batch_smem);
        else if (el.m <= 32)
            finish_t<int32_t, 32>(a, el, e, batch_smem);
        else if (el.m <= 48)
            finish_t<int32_t, 48>(a, el, e, batch_smem);
        else
            finish_t<int32_t, 64>(a, el, e, batch_smem);
    } else if (!(el.flags & EF_VAL16))
        finish_t<int32_t>(a, el, e, batch_smem);
    else if (!finish_t<_Float16>(a, el, e, batch_smem))
        finish_t<uint16_t>(a, el, e, batch_smem);
}

__global__ __launch_bounds__(BT, 2) void k_batch(BatchArgs a) {
    __shared__ int32_t sh_item;
    int32_t home = blockIdx.x % QUEUES, tried = 0;  // (thread 0's are used)
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) {
            FW_GLOBAL int32_t *ctr = gmem(a.ctr);
            int32_t t = a.n_items;
            if (__hip_atomic_load(ctr + CTR_ABORT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
                for (; tried < QUEUES; ++tried, home = (home + 1) % QUEUES) {
                    const int32_t k = __hip_atomic_fetch_add(ctr + home * CTR_STRIDE, 1, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT);
                    if (k < a.queue[home + 1] - a.queue[home]) {
                        t = a.queue[home] + k;
                        break;
                    }
                }
            }
            sh_item = t;
        }
        __syncthreads();
        const int32_t t = __builtin_amdgcn_readfirstlane(sh_item);  // uniform: the item and its election load as scalars
        if (t >= a.n_items) return;
        const BItem it = a.items[t];
        const BElec el = a.elec[it.e];
        if (it.kind == IT_SCAN) {
            if (a.dtype32)
                scan_item<int32_t>(a, el, it.a, it.b);
            else
                scan_item<uint16_t>(a, el, it.a, it.b);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __syncthreads();
            if (threadIdx.x == 0)
                __hip_atomic_fetch_add(gmem(a.ctr) + CTR_ELEC + it.e, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if (it.kind == IT_COUNT) {
            count_item(a, el, it.e, it.a, it.b);
        } else {
            finish(a, el, it.e);
        }
    }
}

// Pseudo-random tournament counts for timing the closure schedules:
// d[x][y] + d[y][x] = n for x != y, d[x][x] = 0.
__global__ __launch_bounds__(256) void k_tune_counts(int32_t *d, int32_t E, int32_t m, int32_t n) {
    const int64_t total = (int64_t)E * m * m;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < total; q += (int64_t)gridDim.x * 256) {
        const int64_t e = q / ((int64_t)m * m);
        const int32_t r = (int32_t)(q % ((int64_t)m * m));
        const int32_t x = r / m, y = r % m;
        const int32_t lo = min(x, y), hi = max(x, y);
        uint64_t h = ((uint64_t)e << 40) ^ ((uint64_t)lo << 20) ^ (uint64_t)hi;
        h = (h ^ (h >> 30)) * 0xbf58476d1ce4e5b9ull;
        h = (h ^ (h >> 27)) * 0x94d049bb133111ebull;
        h ^= h >> 31;
        const int32_t v = (int32_t)(h % (uint64_t)(n + 1));
        d[q] = x == y ? 0 : (x < y ? v : n - v);
    }
}

}  // namespace

// ====================================================================== host

struct schulze_batch {
    schulze_ctx *ctx = nullptr;
    int device = 0;
    int32_t E = 0;
    int ballot_dtype = SCHULZE_U16;
    int mode = SCHULZE_WINNING_VOTES;
    bool closure_only = false;
    int32_t topk = 0;
    std::vector<BElec> elec;
    BElec *elec_dev = nullptr;
    BItem *items_full = nullptr, *items_closure = nullptr;
    int32_t queue_full[QUEUES + 1] = {}, queue_closure[QUEUES + 1] = {};
    uint32_t *planes = nullptr;
    char *scratch = nullptr;
    int64_t scratch_bytes = 0;
    int32_t grid = 0;
    int32_t *ctr = nullptr;
    // captured graph
    hipStream_t cap = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    BatchArgs key{};
};

namespace {

// REGISTERS while its one barrier per step costs less than the tiles' rounds.
// One election per workgroup, us, REGISTERS / TILED64: 16 bits m = 96:
// 84 / 100, m = 128: 212 / 99; int32 m = 96: 84 / 126, m = 128: 121 / 126
// (larger matrices do not fit its registers).
int default_variant(int bits, int32_t m) {
    return m <= (bits == 16 ? 96 : 128) ? SCHULZE_BATCH_CLOSURE_REGISTERS : SCHULZE_BATCH_CLOSURE_TILED64;
}

bool variant_ok(int bits, int32_t m, int variant) {
    switch (variant) {
        // register budget of one workgroup at two workgroups per CU
        case SCHULZE_BATCH_CLOSURE_REGISTERS: return round_up(m, 32) <= (bits == 16 ? 192 : 128);
        case SCHULZE_BATCH_CLOSURE_TILED32: return bits == 16;
        case SCHULZE_BATCH_CLOSURE_TILED64: return true;
        case SCHULZE_BATCH_CLOSURE_TILED128: return bits == 16;
        default: return false;
    }
}

int resolve_variant(const schulze_ctx *ctx, int bits, int32_t m) {
    const int b = (int)((m - 1) / 32);
    const int v = ctx->batch_variant[bits == 16 ? 0 : 1][b];
    if (v >= 0 && variant_ok(bits, m, v)) return v;
    return default_variant(bits, m);
}

int32_t padded_size(int variant, int32_t m) {
    switch (variant) {
        case SCHULZE_BATCH_CLOSURE_REGISTERS: return (int32_t)round_up(m, 32);
        case SCHULZE_BATCH_CLOSURE_TILED32: return (int32_t)round_up(m, 32);
        case SCHULZE_BATCH_CLOSURE_TILED64: return (int32_t)round_up(m, 64);
        default: return (int32_t)round_up(m, 128);
    }
}

int batch_grid(schulze_ctx *ctx, int32_t *grid) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_batch, BT, 0) != hipSuccess || per_cu < 1)
        return SCHULZE_EDEVICE;
    *grid = per_cu * ctx->num_cus;
    return SCHULZE_OK;
}

void free_plan(schulze_batch *pl) {
    if (!pl) return;
    (void)hipSetDevice(pl->device);
    (void)hipDeviceSynchronize();
    if (pl->exec) (void)hipGraphExecDestroy(pl->exec);
    if (pl->graph) (void)hipGraphDestroy(pl->graph);
    if (pl->cap) (void)hipStreamDestroy(pl->cap);
    for (void *ptr : {(void *)pl->elec_dev, (void *)pl->items_full, (void *)pl->items_closure, (void *)pl->planes,
                      (void *)pl->scratch, (void *)pl->ctr})
        if (ptr) (void)hipFree(ptr);
    delete pl;
}

template <typename T>
int upload(T **dst, const std::vector<T> &src) {
    if (src.empty()) return SCHULZE_OK;
    if (hipMalloc((void **)dst, sizeof(T) * src.size()) != hipSuccess) return SCHULZE_ENOMEM;
    if (hipMemcpy(*dst, src.data(), sizeof(T) * src.size(), hipMemcpyHostToDevice) != hipSuccess)
        return SCHULZE_EDEVICE;
    return SCHULZE_OK;
}

int build_plan(schulze_ctx *ctx, const schulze_election *desc, int32_t E, int ballot_dtype, int mode,
               const schulze_batch_options *opt, int forced_variant, schulze_batch **out) {
    *out = nullptr;
    int32_t max_range = RANGE_PAIRS;
    bool closure_only = false;
    if (opt) {
        if (opt->max_range_pairs < 0) return SCHULZE_EINVAL;
        if (opt->max_range_pairs > 0) max_range = std::min(max_range, opt->max_range_pairs);
        closure_only = opt->closure_only != 0;
        if (opt->topk < 0) return SCHULZE_EINVAL;
    }
    schulze_batch *pl = new (std::nothrow) schulze_batch();
    if (!pl) return SCHULZE_ENOMEM;
    pl->ctx = ctx;
    pl->device = ctx->device;
    pl->E = E;
    pl->ballot_dtype = ballot_dtype;
    pl->mode = mode;
    pl->closure_only = closure_only;
    pl->topk = opt ? opt->topk : 0;
    pl->elec.resize(E);
    std::vector<double> cost(E);
    std::vector<int32_t> runs_of(E), ranges_of(E);
    int64_t pos_words = 0;
    int64_t scratch = 256;
    for (int32_t e = 0; e < E; ++e) {
        const schulze_election &s = desc[e];
        BElec &el = pl->elec[e];
        el = BElec{};
        el.ballot_off = s.ballot_off;
        el.n = s.n;
        el.mat_off = s.mat_off;
        el.vec_off = s.vec_off;
        el.m = s.m;
        el.L = s.L;
        el.nb8 = (int32_t)ceil_div(s.m, 8);
        el.pitch = 8 * el.nb8;
        const bool square = s.L < s.m - 1;
        const bool val16 = s.n <= 65535;
        const int bits = val16 ? 16 : 32;
        el.variant = forced_variant >= 0 ? forced_variant : resolve_variant(ctx, bits, s.m);
        if (!variant_ok(bits, s.m, el.variant)) {
            delete pl;
            return SCHULZE_EINVAL;
        }
        el.mp = padded_size(el.variant, s.m);
        const int64_t pairs = (s.n + 1) / 2;
        const int32_t S = square ? el.nb8 * el.nb8 : el.nb8 * (el.nb8 + 1) / 2;
        el.vs = S <= 64 ? 4 : (S <= 128 ? 2 : 1);
        const int32_t runs = (int32_t)ceil_div(S, BT / el.vs);
        const int32_t nq = el.pitch / 4;
        const int32_t groups = (int32_t)ceil_div(nq, 64);
        el.ng = groups <= 1 ? 1 : (groups <= 2 ? 2 : 4);
        el.bits = rank_bits(std::min(s.L, s.m - 1));
        el.rows = CHUNK_QUADS / el.ng;
        if (el.vs > 1) el.rows = el.rows / el.bits * el.bits;  // whole groups (m <= 120: at most 7 planes of 32 rows)
        el.group_pairs = std::min(16, max_range);
        el.range_groups = max_range / el.group_pairs;
        const int64_t vgroups = ceil_div(s.n, 2 * el.group_pairs);
        const int64_t ranges = ceil_div(vgroups, el.range_groups);
        el.flags = (square ? EF_SQUARE : 0) | (ranges > 1 ? EF_MULTI : 0) | (val16 ? EF_VAL16 : 0) |
                   (s.n == 0 ? EF_ZERO_D : 0);
        el.n_count = (int32_t)(runs * ranges);
        runs_of[e] = runs;
        ranges_of[e] = (int32_t)ranges;
        const int32_t vpb = scan_group_pairs(el.pitch, el.group_pairs);
        el.scan_pairs = (int32_t)std::max<int64_t>(vpb, std::min<int64_t>(pairs, SCAN_WORDS / el.pitch) / vpb * vpb);
        el.n_scan = pairs > 0 ? (int32_t)ceil_div(pairs, el.scan_pairs) : 0;
        el.pos_off = pos_words;
        if (!closure_only) pos_words += vgroups * el.bits * el.pitch;
        const int64_t es = val16 ? 2 : 4;
        scratch = std::max<int64_t>(scratch, round_up(es * el.mp * el.mp, 256));
        cost[e] = closure_only ? (double)el.mp * el.mp * el.mp
                               : (double)vgroups * S * (el.bits + 2) * 64.0 + 4.0 * (double)el.mp * el.mp * el.mp;
    }
    // queue: largest elections first
    std::vector<int32_t> order(E);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return cost[x] > cost[y]; });
    int rc = batch_grid(ctx, &pl->grid);
    // each election to the queue with the least work so far
    std::vector<std::vector<int32_t>> queues(QUEUES);
    double load[QUEUES] = {};
    for (int32_t e : order) {
        const int q = (int)(std::min_element(load, load + QUEUES) - load);
        queues[q].push_back(e);
        load[q] += cost[e];
    }
    std::vector<BItem> full, fin;
    for (int q = 0; q < QUEUES; ++q) {
        const std::vector<int32_t> &of = queues[q];
        const int32_t Eq = (int32_t)of.size();
        if (!closure_only && rc == SCHULZE_OK) {
            // Scans (memory-bound) run ahead of the counts (VALU-bound) by `ahead`
            // elections, so that the two overlap; every scan of an election still
            // precedes its counts in the queue.
            auto push_scans = [&](int32_t e) {
                const BElec &el = pl->elec[e];
                const int64_t pairs = (el.n + 1) / 2;
                for (int64_t k = 0; k < pairs; k += el.scan_pairs)
                    full.push_back(BItem{IT_SCAN, e, (int32_t)k, (int32_t)std::min<int64_t>(el.scan_pairs, pairs - k)});
            };
            int32_t ahead = 0;
            for (int64_t items = 0; ahead < Eq && items < 2 * (int64_t)pl->grid / QUEUES; ++ahead)
                items += pl->elec[of[ahead]].n_count;
            for (int32_t i = 0; i < ahead; ++i) push_scans(of[i]);
            for (int32_t i = 0; i < Eq; ++i) {
                const int32_t e = of[i];
                for (int32_t r = 0; r < ranges_of[e]; ++r)
                    for (int32_t u = 0; u < runs_of[e]; ++u) full.push_back(BItem{IT_COUNT, e, u, r});
                if (i + ahead < Eq) push_scans(of[i + ahead]);
            }
            for (int32_t e : of)
                if (pl->elec[e].n_count == 0) full.push_back(BItem{IT_FINISH, e, 0, 0});
        }
        for (int32_t e : of) fin.push_back(BItem{IT_FINISH, e, 0, 0});
        pl->queue_full[q + 1] = (int32_t)full.size();
        pl->queue_closure[q + 1] = (int32_t)fin.size();
    }

    if (rc == SCHULZE_OK) rc = upload(&pl->elec_dev, pl->elec);
    if (rc == SCHULZE_OK) rc = upload(&pl->items_full, full);
    if (rc == SCHULZE_OK) rc = upload(&pl->items_closure, fin);
    if (rc == SCHULZE_OK && pos_words > 0 &&
        hipMalloc((void **)&pl->planes, sizeof(uint32_t) * (size_t)pos_words) != hipSuccess)
        rc = SCHULZE_ENOMEM;
    pl->scratch_bytes = scratch;
    if (rc == SCHULZE_OK && hipMalloc((void **)&pl->scratch, (size_t)scratch * pl->grid) != hipSuccess)
        rc = SCHULZE_ENOMEM;
    if (rc == SCHULZE_OK && hipMalloc((void **)&pl->ctr, sizeof(int32_t) * (size_t)(CTR_ELEC + 2 * (int64_t)E)) != hipSuccess)
        rc = SCHULZE_ENOMEM;
    if (rc != SCHULZE_OK) {
        (void)hipGetLastError();
        free_plan(pl);
        return rc;
    }
    *out = pl;
    return SCHULZE_OK;
}

// The reset of the counters and the persistent launch (graph-capturable).
int enqueue(schulze_batch *pl, hipStream_t s, const BatchArgs &args) {
    schulze_ctx *ctx = pl->ctx;
    int rc = fill_u32(ctx, s, reinterpret_cast<uint32_t *>(pl->ctr), (size_t)(CTR_ELEC + 2 * (int64_t)pl->E), 0u);
    if (rc != SCHULZE_OK) return rc;
    if (args.n_items == 0) return SCHULZE_OK;
    SCHULZE_LAUNCH(ctx, K_BATCH, s, k_batch<<<dim3((unsigned)pl->grid), dim3(BT), 0, s>>>(args));
    return SCHULZE_OK;
}

bool same_args(const BatchArgs &x, const BatchArgs &y) {
    return x.ballots == y.ballots && x.d == y.d && x.p == y.p && x.is_winner == y.is_winner &&
           x.n_winners == y.n_winners && x.beaten_by == y.beaten_by && x.order == y.order &&
           x.level == y.level && x.topk == y.topk && x.closure_only == y.closure_only && x.err == y.err;
}

}  // namespace

extern "C" int schulze_batch_plan(schulze_ctx *ctx, const schulze_election *elections, int32_t E, int ballot_dtype,
                                  int mode, const schulze_batch_options *opt, schulze_batch **plan) {
    if (!plan) return SCHULZE_EINVAL;
    *plan = nullptr;
    if (!ctx || E < 0 || (E > 0 && !elections)) return SCHULZE_EINVAL;
    if (ballot_dtype != SCHULZE_U16 && ballot_dtype != SCHULZE_I32) return SCHULZE_EINVAL;
    if (mode != SCHULZE_WINNING_VOTES && mode != SCHULZE_MARGIN) return SCHULZE_EINVAL;
    if (E > (1 << 24)) return SCHULZE_EUNSUPPORTED;
    for (int32_t e = 0; e < E; ++e) {
        const schulze_election &s = elections[e];
        if (s.m < 1 || s.m > SCHULZE_BATCH_MAX_M || s.L < 1 || s.L > s.m || s.n < 0) return SCHULZE_EINVAL;
        if (s.ballot_off < 0 || s.mat_off < 0 || s.vec_off < 0) return SCHULZE_EINVAL;
        if (s.n > (int64_t)INT32_MAX) return SCHULZE_EUNSUPPORTED;
    }
    if (bind_device(ctx) != SCHULZE_OK) return SCHULZE_EDEVICE;
    return build_plan(ctx, elections, E, ballot_dtype, mode, opt, -1, plan);
}

extern "C" void schulze_batch_destroy(schulze_batch *plan) { free_plan(plan); }

extern "C" int schulze_batch_run(schulze_ctx *ctx, void *stream, schulze_batch *plan, const void *ballots, int32_t *d,
                                 int32_t *p, uint8_t *is_winner, int32_t *n_winners, int32_t *beaten_by,
                                 int32_t *order, int32_t *level, int flags) {
    if (!ctx || !plan || plan->ctx != ctx || !d || !is_winner) return SCHULZE_EINVAL;
    if (level && plan->topk == 0) return SCHULZE_EINVAL;
    if (flags & ~SCHULZE_BATCH_GRAPH) return SCHULZE_EINVAL;
    const bool closure_only = ballots == nullptr;
    if (!closure_only && plan->closure_only) return SCHULZE_EINVAL;
    if (bind_device(ctx) != SCHULZE_OK) return SCHULZE_EDEVICE;
    hipStream_t s = (hipStream_t)stream;
    BatchArgs args{};
    args.elec = plan->elec_dev;
    args.items = closure_only ? plan->items_closure : plan->items_full;
    std::copy_n(closure_only ? plan->queue_closure : plan->queue_full, QUEUES + 1, args.queue);
    args.n_items = args.queue[QUEUES];
    args.n_elec = plan->E;
    args.ballots = ballots;
    args.dtype32 = plan->ballot_dtype == SCHULZE_I32;
    args.mode = plan->mode;
    args.closure_only = closure_only ? 1 : 0;
    args.planes = plan->planes;
    args.d = d;
    args.p = p;
    args.is_winner = is_winner;
    args.n_winners = n_winners;
    args.beaten_by = beaten_by;
    args.order = order;
    args.level = level;
    args.topk = level ? plan->topk : 0;
    args.ctr = plan->ctr;
    args.scratch = plan->scratch;
    args.scratch_bytes = plan->scratch_bytes;
    args.err = ctx->err;
    if (!(flags & SCHULZE_BATCH_GRAPH)) return enqueue(plan, s, args);

    if (!plan->exec || !same_args(plan->key, args)) {
        if (plan->exec) {
            (void)hipGraphExecDestroy(plan->exec);
            plan->exec = nullptr;
        }
        if (plan->graph) {
            (void)hipGraphDestroy(plan->graph);
            plan->graph = nullptr;
        }
        if (!plan->cap && hipStreamCreateWithFlags(&plan->cap, hipStreamNonBlocking) != hipSuccess)
            return SCHULZE_EDEVICE;
        if (hipStreamBeginCapture(plan->cap, hipStreamCaptureModeThreadLocal) != hipSuccess) return SCHULZE_EDEVICE;
        const bool timing = ctx->timing;
        ctx->timing = false;
        int rc = enqueue(plan, plan->cap, args);
        ctx->timing = timing;
        hipGraph_t g = nullptr;
        const hipError_t ec = hipStreamEndCapture(plan->cap, &g);
        if (rc != SCHULZE_OK || ec != hipSuccess || !g) {
            if (g) (void)hipGraphDestroy(g);
            (void)hipGetLastError();
            return rc != SCHULZE_OK ? rc : SCHULZE_EDEVICE;
        }
        if (hipGraphInstantiate(&plan->exec, g, nullptr, nullptr, 0) != hipSuccess) {
            (void)hipGraphDestroy(g);
            plan->exec = nullptr;
            return SCHULZE_EDEVICE;
        }
        plan->graph = g;
        plan->key = args;
    }
    int tok;
    timing_begin(ctx, K_BATCH, s, &tok);
    const hipError_t e = hipGraphLaunch(plan->exec, s);
    timing_end(ctx, tok, s);
    return e == hipSuccess ? SCHULZE_OK : SCHULZE_EDEVICE;
}

extern "C" int schulze_batch_set_closure(schulze_ctx *ctx, int32_t value_bits, int32_t m_lo, int32_t m_hi,
                                         int32_t variant) {
    if (!ctx || (value_bits != 16 && value_bits != 32)) return SCHULZE_EINVAL;
    if (m_lo < 1 || m_hi < m_lo || m_hi > SCHULZE_BATCH_MAX_M) return SCHULZE_EINVAL;
    if (variant < SCHULZE_BATCH_CLOSURE_AUTO || variant > SCHULZE_BATCH_CLOSURE_TILED128) return SCHULZE_EINVAL;
    for (int32_t m = m_lo; m <= m_hi; ++m)
        if (variant >= 0 && !variant_ok(value_bits, m, variant)) return SCHULZE_EINVAL;
    for (int32_t b = (m_lo - 1) / 32; b <= (m_hi - 1) / 32; ++b)
        ctx->batch_variant[value_bits == 16 ? 0 : 1][b] = (int8_t)variant;
    return SCHULZE_OK;
}

extern "C" int schulze_batch_get_closure(schulze_ctx *ctx, int32_t value_bits, int32_t m, int32_t *variant) {
    if (!ctx || !variant || (value_bits != 16 && value_bits != 32) || m < 1 || m > SCHULZE_BATCH_MAX_M)
        return SCHULZE_EINVAL;
    *variant = resolve_variant(ctx, value_bits, m);
    return SCHULZE_OK;
}

extern "C" int schulze_batch_autotune(schulze_ctx *ctx, void *stream, int32_t value_bits, int32_t m_max,
                                      float *ms) {
    if (!ctx || (value_bits != 16 && value_bits != 32) || m_max < 1 || m_max > SCHULZE_BATCH_MAX_M)
        return SCHULZE_EINVAL;
    if (bind_device(ctx) != SCHULZE_OK) return SCHULZE_EDEVICE;
    hipStream_t s = (hipStream_t)stream;
    int32_t grid = 0;
    int rc = batch_grid(ctx, &grid);
    if (rc != SCHULZE_OK) return rc;
    const int32_t nbk = (int32_t)ceil_div(m_max, 32);
    const int32_t m_top = nbk * 32;
    const int32_t E = grid;  // one election per resident workgroup
    const int32_t n = value_bits == 16 ? 60000 : 1000000;
    int32_t *d = nullptr;
    uint8_t *win = nullptr;
    if (hipMalloc((void **)&d, sizeof(int32_t) * (size_t)E * m_top * m_top) != hipSuccess) return SCHULZE_ENOMEM;
    if (hipMalloc((void **)&win, (size_t)E * m_top) != hipSuccess) {
        (void)hipFree(d);
        return SCHULZE_ENOMEM;
    }
    hipEvent_t t0 = nullptr, t1 = nullptr;
    if (hipEventCreate(&t0) != hipSuccess || hipEventCreate(&t1) != hipSuccess) rc = SCHULZE_EDEVICE;
    const bool timing = ctx->timing;
    ctx->timing = false;
    for (int32_t b = 0; b < nbk && rc == SCHULZE_OK; ++b) {
        const int32_t m = 32 * (b + 1);
        k_tune_counts<<<dim3((unsigned)ctx->num_cus * 4), dim3(256), 0, s>>>(d, E, m, n);
        if ((rc = launch_status()) != SCHULZE_OK) break;
        std::vector<schulze_election> desc(E);
        for (int32_t e = 0; e < E; ++e)
            desc[e] = schulze_election{0, n, m, m, (int64_t)e * m * m, (int64_t)e * m};
        schulze_batch_options opt{};
        opt.closure_only = 1;
        float best = 0.f;
        int best_v = -1;
        for (int v = SCHULZE_BATCH_CLOSURE_REGISTERS; v <= SCHULZE_BATCH_CLOSURE_TILED128 && rc == SCHULZE_OK; ++v) {
            if (ms) ms[b * 4 + v] = -1.f;
            if (!variant_ok(value_bits, m, v)) continue;
            schulze_batch *pl = nullptr;
            if ((rc = build_plan(ctx, desc.data(), E, SCHULZE_U16, SCHULZE_WINNING_VOTES, &opt, v, &pl)) !=
                SCHULZE_OK)
                break;
            float t = 0.f;
            rc = schulze_batch_run(ctx, stream, pl, nullptr, d, nullptr, win, nullptr, nullptr, nullptr, nullptr, 0);
            for (int rep = 0; rep < 2 && rc == SCHULZE_OK; ++rep) {
                float tr = 0.f;
                if (hipEventRecord(t0, s) != hipSuccess) rc = SCHULZE_EDEVICE;
                if (rc == SCHULZE_OK)
                    rc = schulze_batch_run(ctx, stream, pl, nullptr, d, nullptr, win, nullptr, nullptr, nullptr, nullptr, 0);
                if (rc == SCHULZE_OK &&
                    (hipEventRecord(t1, s) != hipSuccess || hipEventSynchronize(t1) != hipSuccess ||
                     hipEventElapsedTime(&tr, t0, t1) != hipSuccess))
                    rc = SCHULZE_EDEVICE;
                t = rep == 0 ? tr : std::min(t, tr);
            }
            free_plan(pl);
            if (rc != SCHULZE_OK) break;
            if (ms) ms[b * 4 + v] = t;
            if (best_v < 0 || t < best) {
                best = t;
                best_v = v;
            }
        }
        if (rc == SCHULZE_OK && best_v >= 0) ctx->batch_variant[value_bits == 16 ? 0 : 1][b] = (int8_t)best_v;
    }
    ctx->timing = timing;
    if (t0) (void)hipEventDestroy(t0);
    if (t1) (void)hipEventDestroy(t1);
    (void)hipStreamSynchronize(s);
    (void)hipFree(d);
    (void)hipFree(win);
    return rc;
}
