// Device helpers shared by the kernels that work on tiles of 16 nodes
// (dss_tile.hip, train.hip): matrix instructions, the spread of units and latent
// components over a wavefront's lanes, sender rows, LDS staging.
#pragma once

#include <hip/hip_runtime.h>

#include "dss_tile.h"

namespace ddmgnn {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

template <typename T>
struct Mx;
template <>
struct Mx<double> {
    using A4 = d4;
    using Chunk = d2;  // 16 bytes
    static constexpr int PER = 2;
    static __device__ __forceinline__ d4 mm(double a, double b, d4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ double relu(double x) { return fmax(x, 0.0); }
};
template <>
struct Mx<float> {
    using A4 = f4;
    using Chunk = f4;
    static constexpr int PER = 4;
    static __device__ __forceinline__ f4 mm(float a, float b, f4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ float relu(float x) { return fmaxf(x, 0.0f); }
};

// Row of a 16-row result held by group g in register r (the instructions' layouts).
template <typename T>
__host__ __device__ constexpr int row_of(int r, int g) {
    return sizeof(T) == 8 ? 4 * r + g : 4 * g + r;
}

// Message unit r of a lane of group g: 0-9 of Phi_out, 10-19 of Phi_in. Units 0-3
// of the four groups are, step by step, four consecutive units of one direction,
// and unit 4 holds the last two of both: a chain over the steps runs in ascending order.
__host__ __device__ constexpr int unit(int g, int r) {
    return r == 0 ? g : r == 1 ? 4 + g : r == 2 ? 10 + g : r == 3 ? 14 + g : g < 2 ? 8 + g : 16 + g;
}
// Latent component in register r of group g (-1: none).
__host__ __device__ constexpr int comp(int g, int r) { return r < 2 ? 4 * r + g : g < 2 ? 8 + g : -1; }

// The lane's values of a blob in LDS.
template <typename T>
struct LaneBlob {
    const T* p;
    int lane;
    __device__ __forceinline__ T operator[](int i) const {
        constexpr int PER = Mx<T>::PER;
        return p[((i / PER) * 64 + lane) * PER + i % PER];
    }
};

// The same of a VtBlob in LDS.
template <typename T, int N, int N_OPS>
struct WeightBlob {
    const T* p;
    int lane;
    __device__ __forceinline__ T operator[](int i) const {
        if (i < N_OPS) return LaneBlob<T>{p, lane}[i];
        return p[VtBlob<T>::ops(N_OPS) + (lane >> 4) * VtBlob<T>::row(N, N_OPS) + (i - N_OPS)];
    }
};

// The lane's values of the 4-row operands at the start of a blob (lane l holds row l % 4 and
// the input of group l / 16, so 16 lanes' values serve all): pairs of operands.
struct QuadBlob {
    const double* p;
    int at;
    __device__ __forceinline__ QuadBlob(const double* blob, int lane) : p(blob), at(lane % 4 + lane / 16 * 4) {}
    __device__ __forceinline__ double operator[](int i) const { return p[(i / 2 * 16 + at) * 2 + i % 2]; }
};

// Sender rows. A row holds 20 values: units 0-3 of the four groups in 16-byte
// pieces (FP32: one per group; FP64: units 0, 1 of every group, then 2, 3), then
// unit 4 of the groups. A lane's five values are spread over its node's row and
// neighbouring lanes serve different nodes, so rows pass through LDS: in global
// memory they are read and written in consecutive pieces by consecutive lanes (five
// times fewer cache accesses than the lanes' own values, which bound the kernel: 182 us
// per block of 85,000 FP32 tiles before, 161 with rows, 115 with the rest below).
constexpr int ROW = 20;
template <typename T>
struct Rows20 {
    static constexpr int PIECES = ROW * (int)sizeof(T) / 16;  // 5 or 10
    static constexpr int EDGES = sizeof(T) == 4 ? 4 : 2;      // edge rows gathered at a time
    static constexpr int RECS = VT_ROWS * VT_TILE;            // edge records read at a time
    static constexpr int LOADS = EDGES * VT_TILE * PIECES / 64;
    static constexpr int BUF = EDGES * VT_TILE * ROW;         // values of a wavefront's buffer
    static_assert(LOADS * 64 == EDGES * VT_TILE * PIECES, "whole loads");
};
template <typename T>
__device__ __forceinline__ void row_get(const T* row, int g, T (&q)[5]) {
    using C = typename Mx<T>::Chunk;
    if constexpr (sizeof(T) == 4) {
        const C v = *reinterpret_cast<const C*>(row + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r) q[r] = v[r];
    } else {
        const C v = *reinterpret_cast<const C*>(row + 2 * g), u = *reinterpret_cast<const C*>(row + 8 + 2 * g);
        q[0] = v[0];
        q[1] = v[1];
        q[2] = u[0];
        q[3] = u[1];
    }
    q[4] = row[16 + g];
}
template <typename T>
__device__ __forceinline__ void row_put(T* row, int g, const T (&q)[5]) {
    using C = typename Mx<T>::Chunk;
    if constexpr (sizeof(T) == 4) {
        *reinterpret_cast<C*>(row + 4 * g) = C{q[0], q[1], q[2], q[3]};
    } else {
        *reinterpret_cast<C*>(row + 2 * g) = C{q[0], q[1]};
        *reinterpret_cast<C*>(row + 8 + 2 * g) = C{q[2], q[3]};
    }
    row[16 + g] = q[4];
}

// Latent state of a tile: 16-byte chunks of consecutive lanes. x4 (FP64): the entry
// Psi takes past the components (c in group 2, the in-degree in group 3).
template <typename T>
__device__ __forceinline__ void store_h(T* H, size_t t, int lane, const T (&h)[3], T x4) {
    using C = typename Mx<T>::Chunk;
    C* p = reinterpret_cast<C*>(H) + t * (64 * 4 / Mx<T>::PER) + lane;
    if constexpr (sizeof(T) == 4) {
        p[0] = C{h[0], h[1], h[2], 0};
    } else {
        p[0] = C{h[0], h[1]};
        p[64] = C{h[2], x4};
    }
}
template <typename T>
__device__ __forceinline__ void load_h(const T* H, size_t t, int lane, T (&h)[3], T& x4) {
    using C = typename Mx<T>::Chunk;
    const C* p = reinterpret_cast<const C*>(H) + t * (64 * 4 / Mx<T>::PER) + lane;
    if constexpr (sizeof(T) == 4) {
        const C v = p[0];
        h[0] = v[0];
        h[1] = v[1];
        h[2] = v[2];
    } else {
        const C v = p[0], u = p[64];
        h[0] = v[0];
        h[1] = v[1];
        h[2] = u[0];
        x4 = u[1];
    }
}

// A value that no kernel writes while this one runs, at an address common to the
// wavefront: a scalar load. (Plain loads beside the kernel's own stores are
// vector loads, and what depends on them counts as different per lane.)
template <typename U>
__device__ __forceinline__ U uload(const U* p) {
    return *(const __attribute__((address_space(4))) U*)p;
}
typedef int i4 __attribute__((ext_vector_type(4)));

// Sixteen bytes per lane from global memory to consecutive LDS addresses (to: uniform).
__device__ __forceinline__ void to_lds(const char* from, char* to) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)from,
                                     (__attribute__((address_space(3))) void*)to, 16, 0, 0);
}
// Copies N values per lane to LDS, a chunk of 1 KB per wavefront at a time.
template <typename T, int N, int BLOCK>
__device__ __forceinline__ void stage(const T* __restrict__ from, T* to) {
    constexpr int CH = N / Mx<T>::PER;
    static_assert(N % Mx<T>::PER == 0, "whole chunks");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
#pragma unroll
    for (int i0 = 0; i0 < CH; i0 += BLOCK / 64)
        if (i0 + wave < CH)
            to_lds(reinterpret_cast<const char*>(from) + (i0 + wave) * 1024 + lane * 16,
                   reinterpret_cast<char*>(to) + (i0 + wave) * 1024);
}

// Loads into LDS have arrived.
__device__ __forceinline__ void vmem_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// Orders a wavefront's own LDS traffic: what it wrote is there, what it read is done.
__device__ __forceinline__ void lds_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

}  // namespace
}  // namespace ddmgnn
