// Ballot rows as aligned 16-byte pieces.  No GPU code beyond the qualifiers: the
// addresses are tested on the CPU.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// Ballot rows in 16-byte pieces whatever their length and alignment: piece j
// of a row is the j-th aligned 16 bytes that hold one of its entries, and
// entry e of it has position j PER + e - head (outside 0 .. L-1: another
// row's).  The few pieces that reach outside the ballot array (its first and
// last, if the array is not aligned) are put together entry by entry; in their
// place every lane loads `spare`, the array's first piece that lies inside, so
// that the loads stay unconditional (an array without one is read entry by
// entry altogether).  LONG: rows of more than 64 entries; the row's second
// piece lies inside the row and stands in, with no further address to keep.
template <bool I32, bool LONG = false>
struct RowPieces {
    static constexpr int SIZE = I32 ? 4 : 2, PER = 16 / SIZE;
    const char *lo, *hi, *at;  // the ballot array, and the row's first piece
    const char *spare;
    int32_t head, count;
    __host__ __device__ RowPieces(const void *ballots, int64_t n, int32_t L, int64_t row) {
        lo = static_cast<const char *>(ballots);
        hi = lo + n * L * SIZE;
        const char *p = lo + row * L * SIZE;
        at = reinterpret_cast<const char *>(reinterpret_cast<uintptr_t>(p) & ~(uintptr_t)15);
        head = (int32_t)(p - at) / SIZE;
        count = (head + L + PER - 1) / PER;
        spare = LONG ? at + 16 : lo + (-reinterpret_cast<uintptr_t>(lo) & 15);
        if (!LONG && hi - spare < 16) spare = nullptr;
    }
    __host__ __device__ const char *piece(int32_t j) const { return at + 16 * (int64_t)(j < count ? j : count - 1); }
    __host__ __device__ bool inside(const char *p) const { return p >= lo && p + 16 <= hi; }
    // what is loaded for the piece at p (if there is a spare)
    __host__ __device__ const char *source(const char *p) const { return inside(p) ? p : spare; }
    // pieces j, j + 64, .. of a lane, in flight together
    template <int FLY>
    __host__ __device__ void load(v4u (&x)[FLY], int32_t j) const {
        if (LONG || spare)
            for (int u = 0; u < FLY; ++u) x[u] = *reinterpret_cast<const v4u *>(source(piece(j + 64 * u)));
        if ((!LONG && !spare) || !inside(at) || !inside(piece(count - 1)))
            for (int u = 0; u < FLY; ++u) {
                const char *p = piece(j + 64 * u);
                if (inside(p)) continue;
                for (int e = 0; e < 4; ++e) {
                    uint32_t w = 0xFFFFFFFFu;
                    for (int h = 0; h < PER / 4; ++h) {
                        const char *q = p + 4 * e + SIZE * h;
                        if (q < lo || q + SIZE > hi) continue;
                        if (I32)
                            w = *reinterpret_cast<const uint32_t *>(q);
                        else
                            w = h ? (w & 0xFFFFu) | ((uint32_t)*reinterpret_cast<const uint16_t *>(q) << 16)
                                  : (w & 0xFFFF0000u) | *reinterpret_cast<const uint16_t *>(q);
                    }
                    x[u][e] = w;
                }
            }
    }
    // f(position, raw id) for the row's entries of piece j
    template <typename F>
    __host__ __device__ void each(const v4u &x, int32_t j, int32_t L, F f) const {
        for (int e = 0; e < PER; ++e) {
            const int32_t t = j * PER + e - head;
            if ((uint32_t)t < (uint32_t)L) f(t, I32 ? x[e] : (e & 1) ? x[e >> 1] >> 16 : x[e >> 1] & 0xFFFFu);
        }
    }
    // the largest id of the piece, padding above all
    __host__ __device__ static uint32_t top(const v4u &x) {
        if constexpr (I32) {
            const uint32_t a = x[0] > x[1] ? x[0] : x[1], b = x[2] > x[3] ? x[2] : x[3];
            return a > b ? a : b;
        }
        typedef unsigned short us2 __attribute__((ext_vector_type(2)));
        const uint32_t w[4] = {x[0], x[1], x[2], x[3]};
        const us2 h = __builtin_elementwise_max(
            __builtin_elementwise_max(__builtin_bit_cast(us2, w[0]), __builtin_bit_cast(us2, w[1])),
            __builtin_elementwise_max(__builtin_bit_cast(us2, w[2]), __builtin_bit_cast(us2, w[3])));
        return h.x > h.y ? h.x : h.y;
    }
};
