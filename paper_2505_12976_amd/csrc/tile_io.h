// 64 x 64 tiles between device memory and LDS, for the passes that need a
// block of a matrix next to its transposed block (edge weights, beats,
// per-candidate statistics).  Interior tiles move as 16-byte vectors (four or
// eight elements per access, so that many bytes are in flight per wavefront),
// whatever the matrix's alignment and pitch: a global access of 16 bytes may
// start at any element, and a row that starts inside a line costs one line
// more per row, not an access per element.  (m = 14187, uint16, an odd pitch:
// edge weights 311 -> 178 us, beaten-by counts 303 -> 155.)  Edge tiles take
// one element per access, clamped into the matrix so that all are in flight.
// 256 threads.
#pragma once

#include "internal.h"

namespace tio {

constexpr int T = 64;       // tile side
constexpr int PITCH = 65;   // LDS row pitch (odd: column reads hit distinct banks)

// 16 bytes at any element's address.
template <typename E>
struct Any16;
template <>
struct Any16<uint16_t> {
    typedef uint32_t type __attribute__((ext_vector_type(4), aligned(2)));
};
template <>
struct Any16<int32_t> {
    typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4)));
};
template <typename E>
__device__ __forceinline__ uint4 load16(const E *p) {
    const typename Any16<E>::type x = *reinterpret_cast<const typename Any16<E>::type *>(p);
    return make_uint4(x[0], x[1], x[2], x[3]);
}
template <typename E>
__device__ __forceinline__ void store16(E *p, const uint4 &v) {
    *reinterpret_cast<typename Any16<E>::type *>(p) = typename Any16<E>::type{v.x, v.y, v.z, v.w};
}
// The same past the caches, for an output larger than they are.
template <typename E>
__device__ __forceinline__ void stream16(E *p, const uint4 &v) {
    __builtin_nontemporal_store(typename Any16<E>::type{v.x, v.y, v.z, v.w},
                                reinterpret_cast<typename Any16<E>::type *>(p));
}

// The V elements of a 16-byte vector.
template <typename E>
__device__ inline void unpack(const uint4 &x, E *e);
template <>
__device__ inline void unpack<int32_t>(const uint4 &x, int32_t *e) {
    e[0] = (int32_t)x.x, e[1] = (int32_t)x.y, e[2] = (int32_t)x.z, e[3] = (int32_t)x.w;
}
template <>
__device__ inline void unpack<uint16_t>(const uint4 &x, uint16_t *e) {
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
    for (int u = 0; u < 4; ++u) {
        e[2 * u] = (uint16_t)(w[u] & 0xFFFFu);
        e[2 * u + 1] = (uint16_t)(w[u] >> 16);
    }
}
template <typename E>
__device__ inline uint4 pack(const E *e);
template <>
__device__ inline uint4 pack<int32_t>(const int32_t *e) {
    return make_uint4((uint32_t)e[0], (uint32_t)e[1], (uint32_t)e[2], (uint32_t)e[3]);
}
template <>
__device__ inline uint4 pack<uint16_t>(const uint16_t *e) {
    uint32_t w[4];
    for (int u = 0; u < 4; ++u) w[u] = (uint32_t)e[2 * u] | ((uint32_t)e[2 * u + 1] << 16);
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// A tile in two halves, so that the loads can be issued early and the LDS
// written later: fetch() loads the tile at (r0, c0) of a rows x cols matrix
// into registers (0 outside), put() writes them to LDS.  VEC (cols a multiple
// of the vector length, so that a vector lies inside or outside): every tile
// takes the same 16-byte loads, vectors outside read the tile's first row or
// vector instead, and what lands outside the matrix is garbage that the caller
// ignores.
template <typename E>
struct Regs {
    static constexpr int PER = T * (T / (16 / (int)sizeof(E))) / 256;  // 16-byte vectors per thread
    uint4 x[PER];
};

template <typename E, bool VEC = false>
__device__ inline void fetch(Regs<E> &g, const E *__restrict__ src, int64_t ld, int32_t r0, int32_t c0, int32_t rows,
                             int32_t cols) {
    constexpr int V = 16 / (int)sizeof(E), VPR = T / V;
    if constexpr (VEC) {
        for (int k = 0; k < Regs<E>::PER; ++k) {
            const int q = threadIdx.x + 256 * k;
            const int32_t r = r0 + q / VPR, c = c0 + (q % VPR) * V;
            g.x[k] = load16<E>(src + (int64_t)(r < rows ? r : r0) * ld + (c < cols ? c : c0));
        }
        return;
    }
    if (r0 + T <= rows && c0 + T <= cols) {
        for (int k = 0; k < Regs<E>::PER; ++k) {
            const int q = threadIdx.x + 256 * k;
            g.x[k] = load16<E>(src + (int64_t)(r0 + q / VPR) * ld + c0 + (q % VPR) * V);
        }
        return;
    }
    E e[Regs<E>::PER][V];
    for (int k = 0; k < Regs<E>::PER; ++k)
        for (int u = 0; u < V; ++u) {
            const int q = threadIdx.x + 256 * k;
            const int32_t r = r0 + q / VPR, c = c0 + (q % VPR) * V + u;
            e[k][u] = src[(int64_t)min(r, rows - 1) * ld + min(c, cols - 1)];
        }
    for (int k = 0; k < Regs<E>::PER; ++k) {
        for (int u = 0; u < V; ++u) {
            const int q = threadIdx.x + 256 * k;
            const int32_t r = r0 + q / VPR, c = c0 + (q % VPR) * V + u;
            e[k][u] = r < rows && c < cols ? e[k][u] : (E)0;
        }
        g.x[k] = pack<E>(e[k]);
    }
}

template <typename E>
__device__ inline void put(E (*t)[PITCH], const Regs<E> &g) {
    constexpr int V = 16 / (int)sizeof(E), VPR = T / V;
    for (int k = 0; k < Regs<E>::PER; ++k) {
        const int q = threadIdx.x + 256 * k;
        E e[V];
        unpack<E>(g.x[k], e);
        for (int u = 0; u < V; ++u) t[q / VPR][(q % VPR) * V + u] = e[u];
    }
}

// t[r][c] = src[(r0 + r) ld + c0 + c], 0 where r0 + r >= rows or c0 + c >= cols.
template <typename E>
__device__ inline void load(E (*t)[PITCH], const E *__restrict__ src, int64_t ld, int32_t r0, int32_t c0,
                            int32_t rows, int32_t cols) {
    Regs<E> g;
    fetch<E>(g, src, ld, r0, c0, rows, cols);
    put<E>(t, g);
}

// dst[(r0 + r) ld + c0 + c] = f(r, c) for r0 + r < rows and c0 + c < cols.
template <typename E, typename F>
__device__ inline void store(E *__restrict__ dst, int64_t ld, int32_t r0, int32_t c0, int32_t rows, int32_t cols,
                             F f) {
    if (r0 + T <= rows && c0 + T <= cols) {
        constexpr int V = 16 / (int)sizeof(E);
        constexpr int VPR = T / V;
        for (int q = threadIdx.x; q < T * VPR; q += 256) {
            const int r = q / VPR, cv = q % VPR;
            E e[V];
            for (int u = 0; u < V; ++u) e[u] = f(r, cv * V + u);
            store16<E>(dst + (int64_t)(r0 + r) * ld + c0 + cv * V, pack<E>(e));
        }
    } else {
        for (int q = threadIdx.x; q < T * T; q += 256) {
            const int r = q / T, c = q % T;
            if (r0 + r < rows && c0 + c < cols) dst[(int64_t)(r0 + r) * ld + c0 + c] = f(r, c);
        }
    }
}

}  // namespace tio
