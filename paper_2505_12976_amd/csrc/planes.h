// Bit planes of ranks, shared by the single-election and the batch counts: 32
// voters per 32-bit word, one word per candidate and bit of the rank.
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

// Bits that hold the ranks 0 .. last and, above every rank that is less
// than `last`, all ones for "not listed".
__host__ __device__ inline int32_t rank_bits(int32_t last) {
    int32_t b = 1;
    while (((1 << b) - 1) < last) ++b;
    return b;
}

// 16 x 16 bit transpose of both halves: bit (16 h + p) of w[b] becomes bit
// (16 h + b) of the old w[p].  The bytes of a pair of words are exchanged by
// two v_perm_b32, the smaller parts by two shifts and two v_bitop3_b32.
__device__ __forceinline__ void transpose16(uint32_t (&w)[16]) {
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const uint32_t a = w[p], b = w[p + 8];
        w[p] = __builtin_amdgcn_perm(b, a, 0x06020400u);      // low bytes of each half: a0 b0 a2 b2
        w[p + 8] = __builtin_amdgcn_perm(b, a, 0x07030501u);  // high bytes: a1 b1 a3 b3
    }
    const uint32_t masks[3] = {0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
    for (int st = 0; st < 3; ++st) {
        const int sh = 4 >> st;
        const uint32_t k = masks[st];
#pragma unroll
        for (int p = 0; p < 16; ++p) {
            if (p & sh) continue;
            const uint32_t a = w[p], b = w[p + sh];
            w[p] = (a & k) | ((b << sh) & ~k);
            w[p + sh] = ((a >> sh) & k) | (b & ~k);
        }
    }
}

// Bits of the `live` first voters of a group (voter 2p + h at bit 16 h + p).
__device__ __forceinline__ uint32_t voter_bits(int32_t live) {
    return ((1u << ((live + 1) / 2)) - 1u) | (((1u << (live / 2)) - 1u) << 16);
}

// The masks of an 8 x 8 block of candidate pairs, four to a register tuple.
// v_bitop3_b32 issues at twice the rate of most vector instructions (66
// against 37 T lane operations/s measured, 55 and 33 on random data, which
// costs clock) unless its three sources sit in registers of one parity.  The
// column words come in aligned tuples of four (word j in a register of j's
// parity), so the mask of column j is kept in the other parity's place of its
// own tuple; keep() holds the tuples together.
struct Masks {
    typedef uint32_t v4 __attribute__((ext_vector_type(4)));
    v4 t[8][2];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i][0] = t[i][1] = v4{0u, 0u, 0u, 0u};
        keep();
    }
    __device__ __forceinline__ void keep() {
#pragma unroll
        for (int i = 0; i < 8; ++i) asm("" : "+v"(t[i][0]), "+v"(t[i][1]));
    }
    __device__ __forceinline__ uint32_t get(int i, int j) const { return t[i][j >> 2][(j & 3) ^ 1]; }
    // one more bit of the ranks, lowest first: rows x, columns y
    __device__ __forceinline__ void step(const v4 (&x)[2], const v4 (&y)[2]) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) {  // (~x & y) | (~(x ^ y) & lt)
                const int q = (j & 3) ^ 1;
                t[i][j >> 2][q] =
                    __builtin_amdgcn_bitop3_b32(x[i >> 2][i & 3], y[j >> 2][j & 3], t[i][j >> 2][q], 0x8E);
            }
        keep();
    }
    // acc += population counts (the instruction adds: written out, as the
    // compiler splits the addition off)
    __device__ __forceinline__ void count(uint32_t (&acc)[8][8]) const {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 8; ++j) asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(acc[i][j]) : "v"(get(i, j)));
    }
};
