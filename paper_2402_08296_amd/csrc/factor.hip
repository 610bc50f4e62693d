// Device factorisation: the exact local solvers of DDM-LU (eq. (7); the
// paper's comparator of Tables I and III) and the coarse level (Sec. III.A
// step 1). For every sub-mesh i the dense local matrix A_i = R_i A R_i^T is
// assembled from the CSR matrix, and the coarse matrix A_0 = R_0 A R_0^T
// from the CSR matrix and the partition-of-unity weights; both are inverted
// in place, so that every apply is one GEMV per sub-mesh (lu_local_kernel) and
// one for the coarse level (coarse_kernel).
//
// Storage: a symmetric matrix of order k is held as the 64 x 64 tiles of its lower
// triangle (tile (I, J), J <= I, at I (I + 1) / 2 + J, row-major), the last row
// and column of tiles padded with the identity, so no kernel looks at bounds.
//
// Inversion: the blocked symmetric sweep without pivoting, which is safe for a
// symmetric positive definite matrix (every pivot block is a diagonal block of
// a Schur complement, itself SPD). For pivot block P and the other indices R, S
// one step replaces, with D = A_PP^{-1},
//   A_RS <- A_RS - A_RP D A_PS,   A_RP <- A_RP D,   A_PP <- -D,
// which keeps the matrix symmetric, and after the last block it holds -A^{-1}
// (the readers take the sign). Half the tiles of a Gauss-Jordan step on the
// full square, and half the memory.
//
// The batch of the K local matrices takes two launches per pivot step over the
// whole device: the panel A_RP D of every R,
// then the update of every tile of every matrix, in which the workgroup of the
// next pivot block also inverts it while the others update theirs. Products run
// on the FP64 matrix instructions. 300 matrices of about 900 rows: 73 ms for the
// Gauss-Jordan on full squares with vector products and four launches a step, 11 ms now. A workgroup finds its matrix by binary search
// in a prefix of per-matrix workgroup counts; matrices already finished at that
// step return at once.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.h"

namespace ddmgnn {

namespace {

constexpr int GJ_THREADS = 256;
constexpr int GJ_W = SYM_TILE;  // order of a tile and width of a pivot block
constexpr int GJ_N = GJ_W * GJ_W;
static_assert(GJ_W == 64 && GJ_THREADS == 256, "a wavefront per 16 rows of a tile");

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

// Binary search of node g in the ascending slice s[0..k); -1 when absent.
__device__ inline int find_local(const int32_t* __restrict__ s, int k, int32_t g) {
    int lo = 0, hi = k;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (s[mid] < g) lo = mid + 1;
        else hi = mid;
    }
    return lo < k && s[lo] == g ? lo : -1;
}

// A_i = R_i A R_i^T of sub-mesh subs[blockIdx.x] into its (zeroed) tiles.
__global__ __launch_bounds__(GJ_THREADS) void lu_assemble_kernel(LuMatrix a, const int32_t* __restrict__ subs,
                                                                  const int64_t* __restrict__ off,
                                                                  double* __restrict__ inv) {
    const int32_t* __restrict__ rowptr = a.rowptr;
    const int32_t* __restrict__ col = a.col;
    const double* __restrict__ val = a.val;
    const int i = subs[blockIdx.x];
    const int b = a.sub_ptr[i];
    const int k = a.sub_ptr[i + 1] - b;
    double* M = inv + off[blockIdx.x];
    const int32_t* s = a.sub_nodes + b;
    auto at = [&](int r, int c) { return M + sym_tile(r / GJ_W, c / GJ_W) + (r % GJ_W) * GJ_W + c % GJ_W; };
    for (int j = threadIdx.x; j < (k + GJ_W - 1) / GJ_W * GJ_W; j += GJ_THREADS) {
        if (j >= k) {
            *at(j, j) = 1.0;
            continue;
        }
        const int32_t g = s[j];
        for (int32_t e = rowptr[g]; e < rowptr[g + 1]; ++e) {
            const int q = find_local(s, k, col[e]);
            if (q >= 0 && q / GJ_W <= j / GJ_W) *at(j, q) = val[e];
        }
    }
}

// A_0 = Z^T A Z (column i of Z is R_i^T D_i R_i 1): row i sums w_a A[g_a][m] w_b
// over the slots a of sub-mesh i, the nonzeros (g_a, m) of A and the slots b
// of node m (sub-mesh j = slot_sub[b]). One workgroup builds one row. A row has
// few nonzero columns (the sub-meshes that touch sub-mesh i or its neighbours),
// so the workgroup first marks them in an LDS bitmap, then every thread sums a
// contiguous chunk of the slots into its own accumulator per marked column, and
// the chunks' sums are added in thread order: the bits do not depend on
// scheduling. A row with more than CA_MAXJ columns, or K above CA_MAXK, is
// summed by one thread in slot, nonzero and membership order.
constexpr int CA_THREADS = 256;
constexpr int CA_MAXK = 16384;  // columns covered by the LDS bitmap
constexpr int CA_MAXJ = 32;     // nonzero columns per row held in LDS
__global__ __launch_bounds__(CA_THREADS) void coarse_assemble_kernel(const int32_t* __restrict__ rowptr,
                                                                     const int32_t* __restrict__ col,
                                                                     const double* __restrict__ val,
                                                                     const int32_t* __restrict__ sub_ptr,
                                                                     const int32_t* __restrict__ sub_nodes,
                                                                     const double* __restrict__ weights,
                                                                     const int32_t* __restrict__ node_ptr,
                                                                     const int32_t* __restrict__ node_slots,
                                                                     const int32_t* __restrict__ slot_sub, int K,
                                                                     double* __restrict__ a0) {
    __shared__ uint32_t bits[CA_MAXK / 32];
    __shared__ int32_t wpre[CA_MAXK / 32 + 1];
    __shared__ int32_t cols[CA_MAXJ];
    __shared__ double acc[CA_MAXJ][CA_THREADS + 1];
    const int i = blockIdx.x, t = threadIdx.x;
    double* row = a0 + (size_t)i * K;
    for (int j = t; j < K; j += CA_THREADS) row[j] = 0.0;
    const int s0 = sub_ptr[i], s1 = sub_ptr[i + 1];
    if (K <= CA_MAXK) {  // uniform over the workgroup
        const int W = (K + 31) / 32;
        for (int w = t; w < W; w += CA_THREADS) bits[w] = 0u;
        __syncthreads();
        for (int a = s0 + t; a < s1; a += CA_THREADS) {
            if (weights[a] == 0.0) continue;
            const int32_t g = sub_nodes[a];
            for (int32_t e = rowptr[g]; e < rowptr[g + 1]; ++e) {
                const int32_t m = col[e];
                for (int32_t q = node_ptr[m]; q < node_ptr[m + 1]; ++q) {
                    const int32_t j = slot_sub[node_slots[q]];
                    atomicOr(&bits[j >> 5], 1u << (j & 31));
                }
            }
        }
        __syncthreads();
        if (t == 0) {
            int c = 0;
            for (int w = 0; w < W; ++w) {
                wpre[w] = c;
                c += __popc(bits[w]);
            }
            wpre[W] = c;
        }
        __syncthreads();
        const int nj = wpre[W];
        if (nj <= CA_MAXJ) {  // uniform
            for (int w = t; w < W; w += CA_THREADS) {
                uint32_t b = bits[w];
                for (int c = wpre[w]; b; ++c, b &= b - 1u) cols[c] = w * 32 + __ffs((int)b) - 1;
            }
            for (int c = 0; c < nj; ++c) acc[c][t] = 0.0;
            const int per = (s1 - s0 + CA_THREADS - 1) / CA_THREADS;
            const int a_lo = s0 + t * per, a_hi = min(s1, a_lo + per);
            for (int a = a_lo; a < a_hi; ++a) {
                const double wa = weights[a];
                if (wa == 0.0) continue;
                const int32_t g = sub_nodes[a];
                for (int32_t e = rowptr[g]; e < rowptr[g + 1]; ++e) {
                    const int32_t m = col[e];
                    const double v = val[e] * wa;
                    for (int32_t q = node_ptr[m]; q < node_ptr[m + 1]; ++q) {
                        const int32_t b = node_slots[q], j = slot_sub[b];
                        const int c = wpre[j >> 5] + __popc(bits[j >> 5] & ((1u << (j & 31)) - 1u));
                        acc[c][t] += v * weights[b];
                    }
                }
            }
            __syncthreads();
            for (int c = t; c < nj; c += CA_THREADS) {
                double sum = 0.0;
                for (int u = 0; u < CA_THREADS; ++u) sum += acc[c][u];
                row[cols[c]] = sum;
            }
            return;
        }
    }
    __syncthreads();  // the row is zero before the single-thread sum writes it
    if (t != 0) return;
    for (int a = s0; a < s1; ++a) {
        const double wa = weights[a];
        if (wa == 0.0) continue;
        const int32_t g = sub_nodes[a];
        for (int32_t e = rowptr[g]; e < rowptr[g + 1]; ++e) {
            const int32_t m = col[e];
            const double v = val[e] * wa;
            for (int32_t q = node_ptr[m]; q < node_ptr[m + 1]; ++q) {
                const int32_t b = node_slots[q];
                row[slot_sub[b]] += v * weights[b];
            }
        }
    }
}

// Exact symmetry of A_0: both triangles take the mean of the two sums; the
// diagonal is kept in diag0 (the reference of the pivot test).
__global__ __launch_bounds__(256) void coarse_symmetrise_kernel(double* __restrict__ a0, int K,
                                                                double* __restrict__ diag0) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)K * K) return;
    const int i = (int)(e / K), j = (int)(e % K);
    if (j == i) diag0[i] = a0[e];
    if (j <= i) return;
    const double m = 0.5 * (a0[(size_t)i * K + j] + a0[(size_t)j * K + i]);
    a0[(size_t)i * K + j] = m;
    a0[(size_t)j * K + i] = m;
}

// The K x K coarse matrix into nt x nt tiles (one per workgroup, padded with the
// identity), and back.
template <bool PACK>
__global__ __launch_bounds__(GJ_THREADS) void square_tiles_kernel(double* __restrict__ a, int K, int nt,
                                                                 double* __restrict__ tiles) {
    const int I = blockIdx.x / nt, J = blockIdx.x % nt;
    double* T = tiles + (size_t)blockIdx.x * GJ_N;
    for (int e = threadIdx.x; e < GJ_N; e += GJ_THREADS) {
        const int r = I * GJ_W + e / GJ_W, c = J * GJ_W + e % GJ_W;
        const bool in = r < K && c < K;
        if (PACK) T[e] = in ? a[(size_t)r * K + c] : r == c ? 1.0 : 0.0;
        else if (in) a[(size_t)r * K + c] = T[e];
    }
}

struct GjBatch {
    double* base;
    const int64_t* off;     // [nm + 1] matrix m's tiles at base + off[m]
    const int32_t* order;   // [nm] k_m
    const int32_t* rows;    // [nm + 1] prefix of the tiles per column
    const int32_t* tiles;   // [nm + 1] prefix of the tiles
    int nm;
    double* dinv;           // [nm] pivot block inverses
    double* pan;            // per matrix and row of tiles, A_RP before the step
    double* w;              // and A_RP D
    const double* diag0;    // coarse matrix: its original diagonal (pivot test reference), else null
    int* status;            // bit 0: a pivot not positive (or below GJ_REL of diag0)
};
// Matrix of workgroup w in a prefix of per-matrix workgroup counts (the last m
// with prefix[m] <= w), and w's index within that matrix.
__device__ inline int gj_find(const int32_t* prefix, int nm, int w, int* local) {
    int lo = 0, hi = nm;
    while (lo + 1 < hi) {
        const int mid = (lo + hi) >> 1;
        if (prefix[mid] <= w) lo = mid;
        else hi = mid;
    }
    *local = w - prefix[lo];
    return lo;
}

// A pivot is accepted when it is positive and, for the coarse matrix, above
// GJ_REL times its original diagonal entry: a singular or nearly singular A_0
// is refused instead of inverted.
constexpr double GJ_REL = 1e-12;

// A tile in LDS: 16-byte units, unit u of row r at u ^ (r % 32), so that 16 rows'
// equal columns lie on different banks.
__device__ __forceinline__ int swz(int r, int u) { return r * 32 + (u ^ (r & 31)); }
__device__ __forceinline__ double& el(double* t, int r, int c) { return t[swz(r, c / 2) * 2 + c % 2]; }

// A row-major tile from global memory into LDS: straight 16-byte loads.
__device__ __forceinline__ void tile_in(const double* __restrict__ from, double* to) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int p = (i * 4 + wave) * 64 + lane, r = p / 32, u = (p % 32) ^ (r & 31);
        __builtin_amdgcn_global_load_lds(
            (const __attribute__((address_space(1))) void*)(from + r * GJ_W + u * 2),
            (__attribute__((address_space(3))) void*)(to + (i * 4 + wave) * 128), 16, 0, 0);
    }
}
__device__ __forceinline__ void tile_out(double* t, double* __restrict__ to) {
    for (int e = threadIdx.x; e < GJ_N / 2; e += GJ_THREADS) {
        const int r = e / 32, u = e % 32;
        reinterpret_cast<d2*>(to)[e] = reinterpret_cast<const d2*>(t)[swz(r, u)];
    }
}

// The wavefront's 16 rows of L R, every sum in ascending order: entry
// (16 wave + 4 r + g, 16 c + lane % 16) in out[c][r].
__device__ __forceinline__ void product(double* L, double* R, int wave, int lane, d4 (&out)[4]) {
    const int n = lane & 15, g = lane >> 4;
    double a[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) a[s] = el(L, 16 * wave + n, 4 * s + g);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        d4 acc = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 16; ++s)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], el(R, 4 * s + g, 16 * c + n), acc, 0, 0, 0);
        out[c] = acc;
    }
}
// The same of L R^T, group g taking entries 16 g .. 16 g + 15 of the sums: both operands
// are rows, read 16 bytes at a time.
__device__ __forceinline__ void row16(const double* t, int row, int g, double (&v)[16]) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const d2 x = reinterpret_cast<const d2*>(t)[swz(row, 8 * g + s)];
        v[2 * s] = x[0];
        v[2 * s + 1] = x[1];
    }
}
__device__ __forceinline__ void product_rows(const double* L, const double* R, int wave, int lane, d4 (&out)[4]) {
    const int n = lane & 15, g = lane >> 4;
    double a[16];
    row16(L, 16 * wave + n, g, a);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        double b[16];
        row16(R, 16 * c + n, g, b);
        d4 acc = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 16; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], acc, 0, 0, 0);
        out[c] = acc;
    }
}

// Inverse of the tile in LDS (swizzled), handed to out(row, column, value): Gauss-Jordan
// with a wavefront per 16 rows in registers (lane = column); the pivot row passes through
// LDS, one barrier per pivot. first: index of the tile's first row; rows from k on
// are padding with the identity, whose pivots change nothing and are left out. About 0.5 us
// per pivot (2 us with the tile in LDS: two barriers and 16 LDS updates per thread and pivot).
template <class F>
__device__ __forceinline__ void invert_tile(double* t, double (*row)[GJ_W], const double* diag0, int* status,
                                            int first, int k, F out) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    double a[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] = el(t, 16 * wave + r, lane);
    for (int o = 0; o < 4; ++o) {  // pivots of wavefront o
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int q = 16 * o + i;
            if (first + q >= k) break;  // uniform
            if (wave == o) row[i & 1][lane] = a[i];
            __syncthreads();
            const double rq = row[i & 1][lane], dq = row[i & 1][q];
            if (threadIdx.x == 0) {
                const double floor = diag0 ? GJ_REL * fabs(diag0[first + q]) : 0.0;
                if (!(dq > floor) || !isfinite(dq)) atomicOr(status, 1);
            }
            const double piv = 1.0 / dq;
            const bool me = lane == q;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (wave == o && r == i) continue;  // uniform
                union { double d; int w[2]; } f;
                f.d = a[r];
                f.w[0] = __builtin_amdgcn_readlane(f.w[0], q);
                f.w[1] = __builtin_amdgcn_readlane(f.w[1], q);
                const double x = -f.d * piv;
                a[r] = me ? x : fma(x, rq, a[r]);
            }
            if (wave == o) a[i] = me ? piv : rq * piv;
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) out(16 * wave + r, lane, a[r]);
}
// The same into a row-major tile.
__device__ void invert_tile(double* t, double (*row)[GJ_W], const GjBatch& b, int first, int k,
                            double* __restrict__ inv) {
    invert_tile(t, row, b.diag0, b.status, first, k, [&](int r, int c, double v) { inv[r * GJ_W + c] = v; });
}

// (R_i A R_i^T)^{-1} of a sub-mesh of at most one tile, as a square of even row stride:
// assembled and inverted in LDS, four threads per row of the matrix.
__global__ __launch_bounds__(GJ_THREADS) void lu_small_kernel(LuMatrix a, const int32_t* __restrict__ subs,
                                                             const int64_t* __restrict__ lu_off,
                                                             double* __restrict__ inv, int* status) {
    __shared__ __align__(16) double t[GJ_N];
    __shared__ double row[2][GJ_W];
    __shared__ int32_t nodes[GJ_W];
    const int i = subs[blockIdx.x], b = a.sub_ptr[i], k = a.sub_ptr[i + 1] - b;
    for (int e = threadIdx.x; e < GJ_N; e += GJ_THREADS) t[e] = 0.0;
    if ((int)threadIdx.x < k) nodes[threadIdx.x] = a.sub_nodes[b + threadIdx.x];
    __syncthreads();
    const int j = threadIdx.x / 4;
    if (j < k) {
        const int32_t g = nodes[j], e1 = a.rowptr[g + 1];
        for (int32_t e = a.rowptr[g] + threadIdx.x % 4; e < e1; e += 4) {
            const int q = find_local(nodes, k, a.col[e]);
            if (q >= 0) el(t, j, q) = a.val[e];
        }
    } else if (threadIdx.x % 4 == 0) {
        el(t, j, j) = 1.0;
    }
    __syncthreads();
    const int ld = (k + 1) & ~1;
    double* const M = inv + lu_off[i];
    invert_tile(t, row, nullptr, status, 0, k, [&](int r, int c, double v) {
        if (r < k && c < ld) M[r * ld + c] = c < k ? v : 0.0;
    });
}

// Squares of the inverses from their tiles (which hold the negative): workgroup (x, y) takes
// tile y of matrix x, transposed through LDS where the square holds it twice.
__global__ __launch_bounds__(GJ_THREADS) void lu_pack_kernel(const int32_t* __restrict__ sub_ptr,
                                                            const int32_t* __restrict__ subs,
                                                            const int64_t* __restrict__ off,
                                                            const double* __restrict__ base,
                                                            const int64_t* __restrict__ lu_off,
                                                            double* __restrict__ inv) {
    __shared__ double t[GJ_W][GJ_W + 1];
    const int i = subs[blockIdx.x], k = sub_ptr[i + 1] - sub_ptr[i], ld = (k + 1) & ~1;
    int I = 0, J = blockIdx.y;
    while (J > I) J -= ++I;
    if (I * GJ_W >= k) return;
    const double* T = base + off[blockIdx.x] + sym_tile(I, J);
    double* M = inv + lu_off[i];
    for (int e = threadIdx.x; e < GJ_N; e += GJ_THREADS) t[e / GJ_W][e % GJ_W] = -T[e];
    __syncthreads();
    auto put = [&](int r, int c, double v) {
        if (r < k && c < ld) M[r * ld + c] = c < k ? v : 0.0;
    };
    for (int e = threadIdx.x; e < GJ_N; e += GJ_THREADS) {
        const int r = e / GJ_W, c = e % GJ_W;
        put(I * GJ_W + r, J * GJ_W + c, t[r][c]);
        if (I != J) put(J * GJ_W + r, I * GJ_W + c, t[c][r]);
    }
}

// The first pivot block of every matrix.
__global__ __launch_bounds__(GJ_THREADS) void gj_first_kernel(GjBatch b) {
    __shared__ __align__(16) double t[GJ_N];
    __shared__ double row[2][GJ_W];
    const int m = blockIdx.x;
    if (b.order[m] <= 0) return;
    tile_in(b.base + b.off[m], t);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    invert_tile(t, row, b, 0, b.order[m], b.dinv + (size_t)m * GJ_N);
}

// Panel of pivot block p: W_R = A_RP D, written to the panel buffer and to the matrix,
// the old A_RP to the other panel buffer; -D to the pivot block.
__global__ __launch_bounds__(GJ_THREADS, 2) void gj_panel_kernel(GjBatch b, int p) {
    __shared__ __align__(16) double x[GJ_N], y[GJ_N];
    int R = 0;
    const int m = gj_find(b.rows, b.nm, blockIdx.x, &R);
    const int nt = b.rows[m + 1] - b.rows[m];
    if (p >= nt) return;
    double* M = b.base + b.off[m];
    const double* D = b.dinv + (size_t)m * GJ_N;
    if (R == p) {
        double* T = M + sym_tile(p, p);
        for (int e = threadIdx.x; e < GJ_N; e += GJ_THREADS) T[e] = -D[e];
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    tile_in(D, y);
    double* T = M + (R > p ? sym_tile(R, p) : sym_tile(p, R));
    if (R > p) {
        tile_in(T, x);
    } else {  // A_RP is the transpose of the stored tile
        for (int e = threadIdx.x; e < GJ_N; e += GJ_THREADS) el(x, e % GJ_W, e / GJ_W) = T[e];
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const size_t at = ((size_t)b.rows[m] + R) * GJ_N;
    tile_out(x, b.pan + at);
    d4 w[4];
    product_rows(x, y, wave, lane, w);  // D is symmetric
    __syncthreads();
    const int n = lane & 15, g = lane >> 4;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) el(x, 16 * wave + 4 * r + g, 16 * c + n) = w[c][r];
    __syncthreads();
    tile_out(x, b.w + at);
    if (R > p) {
        tile_out(x, T);
    } else {
        for (int e = threadIdx.x; e < GJ_N; e += GJ_THREADS) T[e] = el(x, e % GJ_W, e / GJ_W);
    }
}

// A_RS -= W_R A_SP^T on one tile per workgroup; the workgroup of the next pivot block
// (the first of its matrix) also inverts it. Bound by the matrix instructions: 256
// products of 16 x 16 x 4 a tile (32 KB read, 16 KB from the panels' cache lines).
__global__ __launch_bounds__(GJ_THREADS, 2) void gj_update_kernel(GjBatch b, int p) {
    __shared__ __align__(16) double x[GJ_N], y[GJ_N];
    __shared__ double row[2][GJ_W];
    int t = 0;
    const int m = gj_find(b.tiles, b.nm, blockIdx.x, &t);
    const int nt = b.rows[m + 1] - b.rows[m];
    if (p >= nt) return;
    const int next = p + 1 < nt ? (p + 1) * (p + 2) / 2 + p + 1 : 0;  // tile (p + 1, p + 1) changes place with tile 0
    t = t == 0 ? next : t == next ? 0 : t;
    int R = (int)((sqrt(8.0 * t + 1.0) - 1.0) * 0.5);
    while ((R + 1) * (R + 2) / 2 <= t) ++R;
    while (R * (R + 1) / 2 > t) --R;
    const int S = t - R * (R + 1) / 2;
    if (R == p || S == p) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    tile_in(b.w + ((size_t)b.rows[m] + R) * GJ_N, x);
    tile_in(b.pan + ((size_t)b.rows[m] + S) * GJ_N, y);
    const int n = lane & 15, g = lane >> 4;
    double* T = b.base + b.off[m] + sym_tile(R, S);
    double old[4][4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) old[c][r] = T[(16 * wave + 4 * r + g) * GJ_W + 16 * c + n];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    d4 w[4];
    product_rows(x, y, wave, lane, w);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            old[c][r] -= w[c][r];
            T[(16 * wave + 4 * r + g) * GJ_W + 16 * c + n] = old[c][r];
        }
    if (R == p + 1 && S == R) {  // uniform over the workgroup
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) el(x, 16 * wave + 4 * r + g, 16 * c + n) = old[c][r];
        __syncthreads();
        invert_tile(x, row, b, R * GJ_W, b.order[m], b.dinv + (size_t)m * GJ_N);
    }
}

// The coarse matrix is inverted on its full square of tiles, by the Gauss-Jordan step
//   A_IJ <- A_IJ - A_IP D A_PJ,  A_PJ <- D A_PJ,  A_IP <- -A_IP D,  A_PP <- D
// with every sum in ascending order: its bits then do not depend on the tiling or the
// kernel, which matters because solves with the FP32 and BF16 forward round what it
// gives (one flipped rounding of a residual moves such a solution by 1e-8). It is one
// small matrix: half the tiles would save less than a launch.
struct SquareArgs {
    double* tiles;
    int nt, K;
    double* dinv;
    double* row;   // D A_PJ of every J
    double* col;   // A_IP of every I before the step
    GjBatch b;     // status and diag0 of the pivot test
};

__global__ __launch_bounds__(GJ_THREADS) void square_first_kernel(SquareArgs a) {
    __shared__ __align__(16) double t[GJ_N];
    __shared__ double row[2][GJ_W];
    tile_in(a.tiles, t);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    invert_tile(t, row, a.b, 0, a.K, a.dinv);
}

// Workgroup j: A_Pj <- D A_Pj; workgroup nt + i: A_iP <- -A_iP D (i = P: the pivot block).
__global__ __launch_bounds__(GJ_THREADS, 2) void square_panel_kernel(SquareArgs a, int p) {
    __shared__ __align__(16) double x[GJ_N], y[GJ_N];
    const bool rows = (int)blockIdx.x < a.nt;
    const int i = (int)blockIdx.x % a.nt;
    double* T = a.tiles + ((size_t)(rows ? p : i) * a.nt + (rows ? i : p)) * GJ_N;
    if (i == p) {
        if (!rows)
            for (int e = threadIdx.x; e < GJ_N; e += GJ_THREADS) T[e] = a.dinv[e];
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    tile_in(T, x);
    tile_in(a.dinv, y);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    d4 w[4];
    if (rows) {
        product(y, x, wave, lane, w);
    } else {
        tile_out(x, a.col + (size_t)i * GJ_N);
        product(x, y, wave, lane, w);
    }
    const int n = lane & 15, g = lane >> 4;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = (16 * wave + 4 * r + g) * GJ_W + 16 * c + n;
            T[e] = rows ? w[c][r] : -w[c][r];
            if (rows) a.row[(size_t)i * GJ_N + e] = w[c][r];
        }
}

__global__ __launch_bounds__(GJ_THREADS, 2) void square_update_kernel(SquareArgs a, int p) {
    __shared__ __align__(16) double x[GJ_N], y[GJ_N];
    __shared__ double row[2][GJ_W];
    const int nt = a.nt, next = p + 1 < nt ? (p + 1) * (nt + 1) : 0;
    int t = blockIdx.x;
    t = t == 0 ? next : t == next ? 0 : t;  // the next pivot block first
    const int I = t / nt, J = t % nt;
    if (I == p || J == p) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    tile_in(a.col + (size_t)I * GJ_N, x);
    tile_in(a.row + (size_t)J * GJ_N, y);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    d4 w[4];
    product(x, y, wave, lane, w);
    const int n = lane & 15, g = lane >> 4;
    double* T = a.tiles + (size_t)t * GJ_N;
    const bool pivot = I == p + 1 && J == I;  // uniform over the workgroup
    if (pivot) __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = 16 * wave + 4 * r + g, j = 16 * c + n;
            const double v = T[i * GJ_W + j] - w[c][r];
            T[i * GJ_W + j] = v;
            if (pivot) el(x, i, j) = v;
        }
    if (pivot) {
        __syncthreads();
        invert_tile(x, row, a.b, I * GJ_W, a.K, a.dinv);
    }
}

}  // namespace

GjPlan::GjPlan(const std::vector<int32_t>& k) {
    nm = (int)k.size();
    meta.assign((size_t)3 * nm + 2, 0);
    int32_t* rows = meta.data() + nm;
    int32_t* tl = rows + nm + 1;
    for (int m = 0; m < nm; ++m) {
        const int64_t nt = (k[m] + GJ_W - 1) / GJ_W;
        meta[m] = k[m];
        steps = std::max(steps, (int)nt);
        n_rows += nt;
        n_tiles += nt * (nt + 1) / 2;
        rows[m + 1] = (int32_t)std::min<int64_t>(n_rows, INT32_MAX);
        tl[m + 1] = (int32_t)std::min<int64_t>(n_tiles, INT32_MAX);
    }
}

size_t GjPlan::scratch_doubles() const { return ((size_t)nm + 2 * (size_t)n_rows) * GJ_N; }

hipError_t launch_gj_invert(const GjPlan& plan, const int32_t* meta, double* base, const int64_t* off, double* scratch,
                            int* status, hipStream_t s) {
    const int nm = plan.nm;
    if (nm == 0 || plan.n_rows == 0) return hipSuccess;
    if (plan.n_tiles * GJ_THREADS >= (int64_t)1 << 32) return hipErrorInvalidConfiguration;  // grid limit
    double* pan = scratch + (size_t)nm * GJ_N;
    const GjBatch b{base,    off,     meta, meta + nm, meta + 2 * (size_t)nm + 1, nm,
                    scratch, pan,     pan + (size_t)plan.n_rows * GJ_N, nullptr, status};
    hipLaunchKernelGGL(gj_first_kernel, dim3(nm), dim3(GJ_THREADS), 0, s, b);
    for (int p = 0; p < plan.steps; ++p) {
        hipLaunchKernelGGL(gj_panel_kernel, dim3((unsigned)plan.n_rows), dim3(GJ_THREADS), 0, s, b, p);
        hipLaunchKernelGGL(gj_update_kernel, dim3((unsigned)plan.n_tiles), dim3(GJ_THREADS), 0, s, b, p);
    }
    return hipGetLastError();
}

size_t coarse_scratch_doubles(int K) {
    const size_t nt = (size_t)(K + GJ_W - 1) / GJ_W;
    return (nt * nt + 2 * nt + 1) * GJ_N;
}

hipError_t launch_coarse_invert(double* a0, int K, const double* diag0, double* scratch, int* status, hipStream_t s) {
    const int nt = (K + GJ_W - 1) / GJ_W;
    if (nt <= 0) return hipSuccess;
    const size_t sq = (size_t)nt * nt;
    if (sq >= (size_t)1 << 24) return hipErrorInvalidConfiguration;  // grid limit
    GjBatch b{};
    b.diag0 = diag0;
    b.status = status;
    const SquareArgs a{scratch, nt, K, scratch + sq * GJ_N, scratch + (sq + 1) * GJ_N,
                       scratch + (sq + 1 + nt) * GJ_N, b};
    hipLaunchKernelGGL(square_tiles_kernel<true>, dim3((unsigned)sq), dim3(GJ_THREADS), 0, s, a0, K, nt, scratch);
    hipLaunchKernelGGL(square_first_kernel, dim3(1), dim3(GJ_THREADS), 0, s, a);
    for (int p = 0; p < nt; ++p) {
        hipLaunchKernelGGL(square_panel_kernel, dim3(2 * nt), dim3(GJ_THREADS), 0, s, a, p);
        if (nt > 1) hipLaunchKernelGGL(square_update_kernel, dim3((unsigned)sq), dim3(GJ_THREADS), 0, s, a, p);
    }
    hipLaunchKernelGGL(square_tiles_kernel<false>, dim3((unsigned)sq), dim3(GJ_THREADS), 0, s, a0, K, nt, scratch);
    return hipGetLastError();
}

hipError_t launch_lu_assemble(const LuMatrix& a, const int32_t* subs, int n, const int64_t* off, double* base,
                              hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(lu_assemble_kernel, dim3(n), dim3(GJ_THREADS), 0, s, a, subs, off, base);
    return hipGetLastError();
}

hipError_t launch_lu_small(const LuMatrix& a, const int32_t* subs, int n, const int64_t* lu_off, double* out,
                           int* status, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(lu_small_kernel, dim3(n), dim3(GJ_THREADS), 0, s, a, subs, lu_off, out, status);
    return hipGetLastError();
}

hipError_t launch_lu_pack(const int32_t* sub_ptr, const int32_t* subs, int n, const int64_t* off, const double* base,
                          const int64_t* lu_off, double* out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    constexpr int NT = (LU_DENSE_K + GJ_W - 1) / GJ_W;
    hipLaunchKernelGGL(lu_pack_kernel, dim3(n, NT * (NT + 1) / 2), dim3(GJ_THREADS), 0, s, sub_ptr, subs, off, base,
                       lu_off, out);
    return hipGetLastError();
}

hipError_t launch_coarse_assemble(const int32_t* rowptr, const int32_t* col, const double* val,
                                  const int32_t* sub_ptr, const int32_t* sub_nodes, const double* weights,
                                  const int32_t* node_ptr, const int32_t* node_slots, const int32_t* slot_sub, int K,
                                  double* a0, double* diag0, hipStream_t s) {
    if (K <= 0) return hipSuccess;
    hipLaunchKernelGGL(coarse_assemble_kernel, dim3(K), dim3(CA_THREADS), 0, s, rowptr, col, val, sub_ptr,
                       sub_nodes, weights, node_ptr, node_slots, slot_sub, K, a0);
    const int64_t kk = (int64_t)K * K;
    hipLaunchKernelGGL(coarse_symmetrise_kernel, dim3((unsigned)((kk + 255) / 256)), dim3(256), 0, s, a0, K, diag0);
    return hipGetLastError();
}

}  // namespace ddmgnn
