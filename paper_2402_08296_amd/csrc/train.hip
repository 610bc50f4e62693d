// Training of DSS_theta (Sec. III.B, Sec. IV.B): the loss is the residual loss
// L_res of Sec. II.B (squared residual of the local system A_i u = c) of the
// decoded state of every block, summed over the kbar blocks.
//
// Work is spread in tiles of 16 nodes over all samples (tile.h: node l % 16 and
// group l / 16 of lane l, five message units and three latent components per
// lane), one launch per block. One workgroup per sample, as before, left the chip
// to as many compute units as samples and every phase to global-memory latency:
// 17.8 ms for 100 samples of 900 nodes, and the same for 17; now 2.00 and 0.89 ms.
//   forward    block b: message sums, Psi, H^{b+1}, the next sender rows, and the
//              decoded state r of H^{b+1}; every block's state, sums and sender
//              rows are kept.
//   residual   rho = A r - c and dL/dr = 2 A rho of all blocks at once (A is
//              symmetric): they do not depend on each other.
//   backward   launch b: the edges of block b + 1 (whose rows the previous launch
//              wrote), then the decoder, Psi and the second message layers of block b.
//
// Weight gradients are sums over the nodes of outer products of per-node
// values. The per-edge terms of the first message layer reduce to per-node
// sums first: with g_e the gradient of edge e's hidden pre-activation (the
// receiver's back-propagated message gradient masked by the edge's ReLU),
//   dW1[:, h_j] = sum_j (sum_{e into j} g_e) h_j^T,
//   dW1[:, h_l] = sum_l (sum_{e out of l} g_e) h_l^T,
// and the coordinate and |d| columns take sums of g_e d_e and g_e |d_e|. A
// wavefront contracts each tile's values over its nodes by matrix products
// into accumulators that it keeps over all its tiles; the wavefronts of a
// workgroup, then the workgroups (in FP64), are added in a fixed order, so the
// gradient is deterministic.
// Arithmetic is FP32; the matrix instruction is a chain of fused multiply-adds
// in ascending input order, so forward values are those of a scalar loop, a
// recomputed pre-activation has the bits of the first evaluation, and the ReLU
// masks agree between the receiver and the sender passes.
#include <algorithm>
#include <cmath>

#include "device.h"
#include "tile.h"

namespace ddmgnn {

namespace {

constexpr int TB = TRAIN_BLOCK;
constexpr int F_PHI = 2 * D + 3, F_PSI = 3 * D + 1;
constexpr int O_PI = D * F_PHI + D + D * D + D;
constexpr int O_PS = 2 * O_PI;
constexpr int O_DE = O_PS + D * F_PSI + D + D * D + D;
static_assert(O_DE + D * D + D + D + 1 == TRAIN_NWB, "weights per block");

// A block's weights as the lanes use them: the three blobs of the FP32 forward,
// then the transposed layers of the backward pass (values per lane).
using L = VtLayout<float>;
constexpr int B_DV = 0, B_DT = 3, B_P2 = 6, B_GH = 9, B_GO = 12, B_GI = 15, B_M16 = 18, B_M4 = 24, N_BACK = 32;
constexpr int E_WX = 0, E_WY = 5, E_WN = 10, E_T1 = 15, E_T2 = 20, N_EDGE = 28;
constexpr int AT_SENDER = L::N_MAIN * 64, AT_DEC = AT_SENDER + L::N_Q * 64, AT_BACK = AT_DEC + L::N_DEC * 64,
              AT_EDGE = AT_BACK + N_BACK * 64, BLOB = AT_EDGE + N_EDGE * 64;
static_assert(BLOB == TRAIN_BLOB, "training blob");

// A backward wavefront's accumulators: matrix products (rows x columns)
//   0-2  [GR 20, GS 20] x [H, 1]            (edges of a block)
//   3    gz x [H, c, 1, fo 0-3]   4  gz x [fo 4-9, fi]
//   5    gfo x [Mo, deg]          6  gfi x [Mi, deg]
//   7    gps x [up, 1]            8  gzd x [H', 1]
// then sums per lane: g dx, g dy, g |d| of its units; dL/dr ud of its components; dL/dr.
constexpr int N_PROD = 9, A_DX = 4 * N_PROD, A_DY = A_DX + 5, A_N = A_DY + 5, A_UD = A_N + 5, A_GR = A_UD + 3,
              N_ACC = A_GR + 2;  // (one unused: whole workgroups in the sums)
static_assert(N_ACC == TRAIN_ACC, "accumulators");

constexpr int EB = 512;             // threads of the forward and backward kernels
constexpr int EW = EB / 64;
constexpr int PG = 2 * ROW;         // receiver part and message gradient of a node, gathered by its senders
constexpr int SR = VT_TILE + 4;     // row stride of a tile's values staged by component
constexpr int N_STAGED = 122;       // rows of the largest staging
constexpr int POOL = 2560;          // floats of a wavefront's buffer: gathered rows, then staged values
static_assert(N_STAGED * SR <= POOL && 2 * VT_TILE * PG <= POOL && 4 * VT_TILE * ROW <= POOL, "wavefront buffer");
constexpr int RECS = VT_ROWS * VT_TILE;

__device__ inline size_t h_at(const TrainArgs& a, int b, size_t t) { return ((size_t)b * a.n_tiles + t) * 256; }
__device__ inline size_t q_at(const TrainArgs& a, int b) { return (size_t)b * (a.n_tiles * VT_TILE + 1) * ROW; }
__device__ inline size_t m_at(const TrainArgs& a, int b) { return (size_t)b * a.n_tiles * 320; }

// Edge records of VT_ROWS rows, in steps of 1 KB.
__device__ __forceinline__ void read_edges(const TrainEdge* from, TrainEdge* to, int lane) {
#pragma unroll
    for (int i = 0; i < RECS * (int)sizeof(TrainEdge) / 1024; ++i)
        to_lds(reinterpret_cast<const char*>(from) + i * 1024 + lane * 16, reinterpret_cast<char*>(to) + i * 1024);
}

// Rows of `PIECES` 16-byte pieces of the edges from row e on (ROWS edge rows) into LDS.
// Records from row `left` on are another tile's: they are not looked at.
template <int PIECES, int ROWS>
__device__ __forceinline__ void gather_rows(const float* rows, const TrainEdge* recs, int e, int left, int delta,
                                            int sentinel, float* to, int lane) {
    constexpr int LOADS = ROWS * VT_TILE * PIECES / 64;
    static_assert(LOADS * 64 == ROWS * VT_TILE * PIECES, "whole loads");
    int l[LOADS];
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int at = e * VT_TILE + (i * 64 + lane) / PIECES;
        l[i] = at < left * VT_TILE ? recs[at].node : -1;
    }
    lds_done();  // also: the buffer's previous rows have been read
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const size_t row = (size_t)(l[i] < 0 ? sentinel : l[i] + delta);
        to_lds(reinterpret_cast<const char*>(rows) + row * (PIECES * 16) + (i * 64 + lane) % PIECES * 16,
               reinterpret_cast<char*>(to) + i * 1024);
    }
}

// Hidden pre-activation of the lane's unit r for one edge: the parts' sum, then the
// coordinate and length terms (Phi_in sees -d).
__device__ __forceinline__ float pre(float pr, float qs, float wx, float wy, float wn, int r, int g, float dx,
                                     float dy, float nd) {
    const bool in = r == 2 || r == 3 || (r == 4 && g >= 2);
    float t = pr + qs;
    t = fmaf(wx, in ? -dx : dx, t);
    t = fmaf(wy, in ? -dy : dy, t);
    return fmaf(wn, nd, t);
}

// A lane's values of its node by component or unit, staged as rows of a tile's 16 nodes.
__device__ __forceinline__ void put_comps(float* st, int row, int n, int g, const float (&v)[3]) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
        if (r < 2 || g < 2) st[(row + comp(g, r)) * SR + n] = v[r];
}
__device__ __forceinline__ void put_units(float* st, int row, int n, int g, const float (&v)[5]) {
#pragma unroll
    for (int r = 0; r < 5; ++r) st[(row + unit(g, r)) * SR + n] = v[r];
}
// Operand of a contraction over the tile's nodes: row of the lane's index, nodes 4g..4g+3.
__device__ __forceinline__ f4 staged(const float* st, int row, int g) {
    return *reinterpret_cast<const f4*>(st + row * SR + 4 * g);
}
__device__ __forceinline__ f4 contract(f4 a, f4 b, f4 c) {
#pragma unroll
    for (int s = 0; s < 4; ++s) c = Mx<float>::mm(a[s], b[s], c);
    return c;
}

// Receiver part b1 + W1[:, h_j] h of the lane's units.
template <class W>
__device__ __forceinline__ void receiver_part(const W& w, const float (&h)[3], float (&p)[5]) {
    f4 acc = {w[L::CP], w[L::CP + 1], w[L::CP + 2], w[L::CP + 3]};
    f4 acc4 = {w[L::CP4], 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        acc = Mx<float>::mm(w[L::P16 + s], h[s], acc);
        acc4 = Mx<float>::mm(w[L::P4 + s], h[s], acc4);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = acc[r];
    p[4] = acc4[0];
}
// Messages fo, fi from their hidden sums, and Psi's hidden pre-activation.
template <class W>
__device__ __forceinline__ void psi_hidden(const W& w, const float (&h)[3], const float (&m)[5], float c, float deg,
                                           int g, f4& fo, f4& fi, f4& z) {
    fo = f4{w[L::CCO] * deg, w[L::CCO + 1] * deg, w[L::CCO + 2] * deg, 0};
    fi = f4{w[L::CCI] * deg, w[L::CCI + 1] * deg, w[L::CCI + 2] * deg, 0};
    z = f4{w[L::CH], w[L::CH + 1], w[L::CH + 2], 0};
    // (entries against zero weights are zeroed, as in dss_block_kernel)
    const float m4o = g < 2 ? m[4] : 0.0f, m4i = g < 2 ? 0.0f : m[4];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        fo = Mx<float>::mm(w[L::FO + s], s < 2 ? m[s] : m4o, fo);
        fi = Mx<float>::mm(w[L::FI + s], s < 2 ? m[2 + s] : m4i, fi);
    }
    fo[2] = g < 2 ? fo[2] : 0.0f;
    fi[2] = g < 2 ? fi[2] : 0.0f;
    z = Mx<float>::mm(w[L::HID], h[0], z);
    z = Mx<float>::mm(w[L::HID + 1], h[1], z);
    z = Mx<float>::mm(w[L::HID + 2], g == 2 ? c : h[2], z);
#pragma unroll
    for (int s = 0; s < 3; ++s) z = Mx<float>::mm(w[L::HID + 3 + s], fo[s], z);
#pragma unroll
    for (int s = 0; s < 3; ++s) z = Mx<float>::mm(w[L::HID + 6 + s], fi[s], z);
}

// The tiles of a wavefront: contiguous slabs per die, strided over its wavefronts.
struct Walk {
    int it, end, step;
};
__device__ __forceinline__ Walk walk(int n_tiles, int wave) {
    const int die = blockIdx.x % N_XCD;
    return {(int)((int64_t)n_tiles * die / N_XCD) + (int)(blockIdx.x / N_XCD) * EW + wave,
            (int)((int64_t)n_tiles * (die + 1) / N_XCD), (int)(gridDim.x / N_XCD) * EW};
}

__device__ inline double block_sum_d(double v, double* sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    __syncthreads();
    if (lane == 0) sh[w] = v;
    __syncthreads();
    double acc = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < TB / 64; ++i) acc += sh[i];
    return acc;
}

// Gathers every block's weights into the lanes' order (map: signed position + 1, 0: zero).
__global__ __launch_bounds__(256) void train_blob_kernel(const float* __restrict__ theta,
                                                        const int32_t* __restrict__ map, float* __restrict__ blobs) {
    const int e = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
    if (e >= BLOB) return;
    const int m = map[e];
    const float v = m == 0 ? 0.0f : theta[(size_t)b * TRAIN_NWB + (m < 0 ? -m : m) - 1];
    blobs[(size_t)b * BLOB + e] = m < 0 ? -v : v;
}

// Inputs of every tile lane, H^0 = 0, block 0's sender rows (W1[:, h_l] 0 = 0) and the
// sentinel rows: the receiver or sender part -inf, so that no message and no
// gradient passes a missing edge.
__global__ __launch_bounds__(256) void train_init_kernel(TrainArgs a) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const float inf = __builtin_inff();
    if (i < (int64_t)a.kbar * ROW) a.q[q_at(a, (int)(i / ROW)) + (size_t)a.n_tiles * VT_TILE * ROW + i % ROW] = -inf;
    if (i < 2 * PG) {
        const int j = (int)(i % PG);
        const bool p = j < 16 || (j >= 32 && j < 36);
        a.pg[i / PG][(size_t)a.n_tiles * VT_TILE * PG + j] = p ? -inf : 0.0f;
    }
    if (i >= (int64_t)a.n_tiles * VT_TILE) return;
    const int t = (int)(i / VT_TILE), n = (int)(i % VT_TILE);
    const int4 x = a.items[2 * (size_t)t], y = a.items[2 * (size_t)t + 1];
    const int2 nd = a.node[(size_t)x.x * VT_TILE + n];
    const int64_t off = (int64_t)((uint64_t)(uint32_t)y.z | (uint64_t)(uint32_t)y.w << 32);
    a.in[i] = float2{nd.x >= 0 ? a.c[off + (nd.x - a.info[x.x].x)] : 0.0f, (float)nd.y};
    f4* h = reinterpret_cast<f4*>(a.h + h_at(a, 0, (size_t)t));
#pragma unroll
    for (int g = 0; g < 4; ++g) h[g * 16 + n] = f4{0, 0, 0, 0};
    f4* q = reinterpret_cast<f4*>(a.q + (size_t)i * ROW);
#pragma unroll
    for (int p = 0; p < 5; ++p) q[p] = f4{0, 0, 0, 0};
}

// One block forward.
template <bool LAST>
__global__ __launch_bounds__(EB, 4) void train_forward_kernel(TrainArgs a, int b) {
    __shared__ __align__(16) float sw[(L::N_MAIN + L::N_Q + L::N_DEC) * 64];
    __shared__ __align__(16) float buf[EW][4 * VT_TILE * ROW];
    __shared__ __align__(16) TrainEdge recs[EW][RECS];
    const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float* blob = a.blobs + (size_t)b * BLOB;
    stage<float, L::N_MAIN, EB>(blob, sw);
    if (!LAST) stage<float, L::N_Q, EB>(blob + BLOB + AT_SENDER, sw + AT_SENDER);  // of the next block
    stage<float, L::N_DEC, EB>(blob + AT_DEC, sw + AT_DEC);
    const LaneBlob<float> w{sw, lane}, wq{sw + AT_SENDER, lane}, wd{sw + AT_DEC, lane};
    Walk k = walk(a.n_tiles, wave);
    vmem_done();
    __syncthreads();
    const int sentinel = a.n_tiles * VT_TILE;
    for (; k.it < k.end; k.it += k.step) {
        asm volatile("" ::: "memory");  // keeps the weights in LDS
        const size_t t = (size_t)k.it;
        const i4 x = uload(reinterpret_cast<const i4*>(a.items) + 2 * t);
        const TrainEdge* rin = a.rin + (size_t)x[2] * VT_TILE;
        const int delta = x[1], md = x[3];
        read_edges(rin, recs[wave], lane);
        float h[3], unused;
        load_h<float>(a.h + (size_t)b * a.n_tiles * 256, t, lane, h, unused);
        const float2 in = a.in[t * VT_TILE + n];
        float p[5], m[5] = {0, 0, 0, 0, 0};
        receiver_part(w, h, p);
        for (int e0 = 0; e0 < md; e0 += VT_ROWS) {
            if (e0) {
                lds_done();
                read_edges(rin + e0 * VT_TILE, recs[wave], lane);
            }
            vmem_done();
            for (int e = 0; e < VT_ROWS && e0 + e < md; e += 4) {
                gather_rows<5, 4>(a.q + q_at(a, b), recs[wave], e, md - e0, delta, sentinel, buf[wave], lane);
                vmem_done();
#pragma unroll
                for (int i = 0; i < 4; i += 2)
                    if (e0 + e + i < md) {  // uniform; md is even
#pragma unroll
                        for (int f = 0; f < 2; ++f) {
                            const TrainEdge ed = recs[wave][(e + i + f) * VT_TILE + n];
                            float q[5];
                            row_get<float>(buf[wave] + ((i + f) * VT_TILE + n) * ROW, g, q);
#pragma unroll
                            for (int r = 0; r < 5; ++r)
                                m[r] += fmaxf(pre(p[r], q[r], w[L::WX + r], w[L::WY + r], w[L::WN + r], r, g, ed.dx,
                                                  ed.dy, ed.nd), 0.0f);
                        }
                    }
            }
        }
        f4 fo, fi, z;
        psi_hidden(w, h, m, in.x, in.y, g, fo, fi, z);
        f4 out = {w[L::CO], w[L::CO + 1], w[L::CO + 2], 0};
#pragma unroll
        for (int s = 0; s < 3; ++s) out = Mx<float>::mm(w[L::OUT + s], fmaxf(z[s], 0.0f), out);
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const float v = fmaf(a.alpha, out[r], h[r]);
            if (r < 2 || g < 2) h[r] = v;
        }
        store_h<float>(a.h + (size_t)(b + 1) * a.n_tiles * 256, t, lane, h, 0.0f);
        float* M = a.m + m_at(a, b);
        reinterpret_cast<f4*>(M)[t * 64 + lane] = f4{m[0], m[1], m[2], m[3]};
        M[(size_t)a.n_tiles * 256 + t * 64 + lane] = m[4];
        // the decoded state of this block
        f4 dh = {wd[L::CDH], wd[L::CDH + 1], wd[L::CDH + 2], 0};
#pragma unroll
        for (int s = 0; s < 3; ++s) dh = Mx<float>::mm(wd[L::DH + s], h[s], dh);
        f4 r = {wd[L::CDO], 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 3; ++s) r = Mx<float>::mm(wd[L::DO + s], fmaxf(dh[s], 0.0f), r);
        if (g == 0) a.r[(t * VT_TILE + n) * a.ks + b] = r[0];
        if constexpr (!LAST) {
            f4 q4 = {0, 0, 0, 0}, q5 = {0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                q4 = Mx<float>::mm(wq[L::Q16 + s], h[s], q4);
                q5 = Mx<float>::mm(wq[L::Q4 + s], h[s], q5);
            }
            const float q[5] = {q4[0], q4[1], q4[2], q4[3], q5[0]};
            lds_done();
            row_put<float>(buf[wave] + n * ROW, g, q);
            lds_done();
            f4* to = reinterpret_cast<f4*>(a.q + q_at(a, b + 1) + t * (VT_TILE * ROW));
            const f4* from = reinterpret_cast<const f4*>(buf[wave]);
            to[lane] = from[lane];
            if (lane < 16) to[64 + lane] = from[64 + lane];
        }
        lds_done();
    }
}

// y = A x - c (FIRST) or 2 A x of every block (values of a tile lane's blocks are
// consecutive); FIRST also sums y^2 per workgroup.
template <bool FIRST>
__global__ __launch_bounds__(TB) void train_residual_kernel(TrainArgs a, const float* __restrict__ x,
                                                           float* __restrict__ y) {
    __shared__ double red[TB / 64];
    const int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x;
    const int64_t lane = i / a.ks;
    const int b = (int)(i % a.ks);
    double sq = 0.0;
    if (lane < (int64_t)a.n_tiles * VT_TILE && b < a.kbar) {
        const int4 it = a.items[2 * (size_t)(lane / VT_TILE)];
        const int slot = a.node[(size_t)it.x * VT_TILE + lane % VT_TILE].x;
        float v = 0.0f;
        if (slot >= 0) {
            const int base = a.info[it.x].x;
            float acc = 0.0f;
            for (int q = a.lm_ptr[slot]; q < a.lm_ptr[slot + 1]; ++q)
                acc = fmaf(a.lm_val[q], x[(int64_t)(a.pos[base + a.lm_col[q]] + it.y) * a.ks + b], acc);
            v = FIRST ? acc - a.in[lane].x : 2.0f * acc;
        }
        y[i] = v;
        sq = (double)v * (double)v;
    }
    if (FIRST) {
        const double tot = block_sum_d(sq, red);
        if (threadIdx.x == 0) a.sse[blockIdx.x] = tot;
    }
}

// Backward launch b: the edges of block b + 1, then the node-local part of block b.
// EDGES is false in the first launch, NODE in the last. Bound by the chain of a
// tile's loads and about a hundred matrix products with eight wavefronts per
// compute unit (256 registers): 45 us a launch for 5,700 tiles, of which the
// gradient products are 36 of the hundred. Separate launches for the two parts
// take as long (27.5 + 20.4 us), and four out-edge rows at a time spill (59 us).
template <bool EDGES, bool NODE>
__global__ __launch_bounds__(EB, 2) void train_backward_kernel(TrainArgs a, int b) {
    constexpr int S_DEC = L::N_MAIN * 64, S_BACK = S_DEC + L::N_DEC * 64, S_EDGE = S_BACK + N_BACK * 64;
    __shared__ __align__(16) float sw[S_EDGE + N_EDGE * 64];
    __shared__ __align__(16) float pool[EW][POOL];
    __shared__ __align__(16) TrainEdge recs[EW][RECS];
    const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (NODE) {
        const float* blob = a.blobs + (size_t)b * BLOB;
        stage<float, L::N_MAIN, EB>(blob, sw);
        stage<float, L::N_DEC, EB>(blob + AT_DEC, sw + S_DEC);
        stage<float, N_BACK, EB>(blob + AT_BACK, sw + S_BACK);
    }
    if (EDGES) stage<float, N_EDGE, EB>(a.blobs + (size_t)(b + 1) * BLOB + AT_EDGE, sw + S_EDGE);
    const LaneBlob<float> w{sw, lane}, wd{sw + S_DEC, lane}, wb{sw + S_BACK, lane}, we{sw + S_EDGE, lane};
    float acc[N_ACC];
#pragma unroll
    for (int i = 0; i < N_ACC; ++i) acc[i] = 0.0f;
    auto product = [&](int i, f4 l, f4 r) {  // accumulator i += sum over the nodes of l x r
        f4 c = {acc[4 * i], acc[4 * i + 1], acc[4 * i + 2], acc[4 * i + 3]};
        c = contract(l, r, c);
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[4 * i + q] = c[q];
    };
    const f4 zero = {0, 0, 0, 0}, one = {1, 1, 1, 1};
    float* const st = pool[wave];
    Walk k = walk(a.n_tiles, wave);
    vmem_done();
    __syncthreads();
    const int sentinel = a.n_tiles * VT_TILE;
    for (; k.it < k.end; k.it += k.step) {
        asm volatile("" ::: "memory");  // keeps the weights in LDS
        const size_t t = (size_t)k.it;
        const i4 x = uload(reinterpret_cast<const i4*>(a.items) + 2 * t);
        const i4 y = uload(reinterpret_cast<const i4*>(a.items) + 2 * t + 1);
        float hc[3], unused;  // H^{b+1}: output of block b, input of block b + 1
        load_h<float>(a.h + (size_t)(b + 1) * a.n_tiles * 256, t, lane, hc, unused);
        f4* const own = reinterpret_cast<f4*>(a.own) + t * 256 + lane;
        f4 gh = zero;  // dL/dH^{b+1}
        if (EDGES) {
            const TrainEdge* rin = a.rin + (size_t)x[2] * VT_TILE;
            const TrainEdge* rout = a.rout + (size_t)y[0] * VT_TILE;
            const int delta = x[1], mi = x[3], mo = y[1];
            read_edges(rin, recs[wave], lane);
            const float* Q = a.q + q_at(a, b + 1);
            const float* G = a.pg[(b + 1) & 1];
            float p[5], q[5], gm[5], gr[5] = {0, 0, 0, 0, 0}, gs[5] = {0, 0, 0, 0, 0};
            const f4 o0 = own[0], o1 = own[64], o2 = own[128], o3 = own[192];
            const float* qrow = Q + (t * VT_TILE + n) * ROW;
            const f4 q0 = *reinterpret_cast<const f4*>(qrow + 4 * g);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p[r] = o0[r];
                gm[r] = o1[r];
                q[r] = q0[r];
            }
            p[4] = o2[0];
            gm[4] = o2[1];
            q[4] = qrow[16 + g];
            float wx[5], wy[5], wn[5];
#pragma unroll
            for (int r = 0; r < 5; ++r) {
                wx[r] = we[E_WX + r];
                wy[r] = we[E_WY + r];
                wn[r] = we[E_WN + r];
            }
            // in-edges: the node receives
            for (int e0 = 0; e0 < mi; e0 += VT_ROWS) {
                if (e0) {
                    lds_done();
                    read_edges(rin + e0 * VT_TILE, recs[wave], lane);
                }
                vmem_done();
                for (int e = 0; e < VT_ROWS && e0 + e < mi; e += 4) {
                    gather_rows<5, 4>(Q, recs[wave], e, mi - e0, delta, sentinel, st, lane);
                    vmem_done();
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (e0 + e + i < mi) {  // uniform
                            const TrainEdge ed = recs[wave][(e + i) * VT_TILE + n];
                            float qs[5];
                            row_get<float>(st + (i * VT_TILE + n) * ROW, g, qs);
#pragma unroll
                            for (int r = 0; r < 5; ++r) {
                                const float v = pre(p[r], qs[r], wx[r], wy[r], wn[r], r, g, ed.dx, ed.dy, ed.nd) > 0.0f
                                                    ? gm[r] : 0.0f;
                                gr[r] += v;
                                acc[A_DX + r] = fmaf(v, ed.dx, acc[A_DX + r]);
                                acc[A_DY + r] = fmaf(v, ed.dy, acc[A_DY + r]);
                                acc[A_N + r] = fmaf(v, ed.nd, acc[A_N + r]);
                            }
                        }
                }
            }
            // out-edges: the node sends
            for (int e0 = 0; e0 < mo; e0 += VT_ROWS) {
                lds_done();
                read_edges(rout + e0 * VT_TILE, recs[wave], lane);
                vmem_done();
                for (int e = 0; e < VT_ROWS && e0 + e < mo; e += 2) {
                    gather_rows<10, 2>(G, recs[wave], e, mo - e0, delta, sentinel, st, lane);
                    vmem_done();
#pragma unroll
                    for (int i = 0; i < 2; ++i) {  // mo is even
                        const TrainEdge ed = recs[wave][(e + i) * VT_TILE + n];
                        const float* row = st + (i * VT_TILE + n) * PG;
                        const f4 pr = *reinterpret_cast<const f4*>(row + 4 * g);
                        const f4 gv = *reinterpret_cast<const f4*>(row + 16 + 4 * g);
                        const float pr4 = row[32 + g], gv4 = row[36 + g];
#pragma unroll
                        for (int r = 0; r < 5; ++r)
                            gs[r] += pre(r < 4 ? pr[r < 4 ? r : 0] : pr4, q[r], wx[r], wy[r], wn[r], r, g, ed.dx,
                                         ed.dy, ed.nd) > 0.0f ? (r < 4 ? gv[r < 4 ? r : 0] : gv4) : 0.0f;
                    }
                }
            }
            gh = f4{o2[2], o2[3], o3[0], 0};
#pragma unroll
            for (int r = 0; r < 5; ++r) {
                gh = Mx<float>::mm(we[E_T1 + r], gr[r], gh);
                gh = Mx<float>::mm(we[E_T2 + r], gs[r], gh);
            }
            lds_done();
            put_units(st, 0, n, g, gr);
            put_units(st, 20, n, g, gs);
            put_comps(st, 40, n, g, hc);
            lds_done();
            const f4 right = n < 10 ? staged(st, 40 + n, g) : n == 10 ? one : zero;
#pragma unroll
            for (int i = 0; i < 3; ++i) product(i, i < 2 || n < 8 ? staged(st, 16 * i + n, g) : zero, right);
            lds_done();
        }
        if (NODE) {
            float hp[3], m[5];
            load_h<float>(a.h + (size_t)b * a.n_tiles * 256, t, lane, hp, unused);
            const float* M = a.m + m_at(a, b);
            const f4 m4 = reinterpret_cast<const f4*>(M)[t * 64 + lane];
#pragma unroll
            for (int r = 0; r < 4; ++r) m[r] = m4[r];
            m[4] = M[(size_t)a.n_tiles * 256 + t * 64 + lane];
            const float2 in = a.in[t * VT_TILE + n];
            const float dr = a.gr[(t * VT_TILE + n) * a.ks + b];
            // decoder
            f4 zd = {wd[L::CDH], wd[L::CDH + 1], wd[L::CDH + 2], 0};
#pragma unroll
            for (int s = 0; s < 3; ++s) zd = Mx<float>::mm(wd[L::DH + s], hc[s], zd);
            float gzd[3], gps[3], up[3], gz[3];
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                gzd[r] = zd[r] > 0.0f ? wb[B_DV + r] * dr : 0.0f;
                acc[A_UD + r] = fmaf(dr, fmaxf(zd[r], 0.0f), acc[A_UD + r]);
            }
            acc[A_GR] += dr;
#pragma unroll
            for (int s = 0; s < 3; ++s) gh = Mx<float>::mm(wb[B_DT + s], gzd[s], gh);
            // Psi
            f4 fo, fi, z, gu = zero;
            psi_hidden(w, hp, m, in.x, in.y, g, fo, fi, z);
#pragma unroll
            for (int r = 0; r < 3; ++r) gps[r] = a.alpha * gh[r];
#pragma unroll
            for (int s = 0; s < 3; ++s) gu = Mx<float>::mm(wb[B_P2 + s], gps[s], gu);
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                up[r] = fmaxf(z[r], 0.0f);
                gz[r] = z[r] > 0.0f ? gu[r] : 0.0f;
            }
            f4 gfo = zero, gfi = zero, gm16 = zero, gm4 = zero;
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                gh = Mx<float>::mm(wb[B_GH + s], gz[s], gh);
                gfo = Mx<float>::mm(wb[B_GO + s], gz[s], gfo);
                gfi = Mx<float>::mm(wb[B_GI + s], gz[s], gfi);
            }
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                gm16 = Mx<float>::mm(wb[B_M16 + s], gfo[s], gm16);
                gm4 = Mx<float>::mm(wb[B_M4 + s], gfo[s], gm4);
            }
#pragma unroll
            for (int s = 0; s < 3; ++s) {
                gm16 = Mx<float>::mm(wb[B_M16 + 3 + s], gfi[s], gm16);
                gm4 = Mx<float>::mm(wb[B_M4 + 3 + s], gfi[s], gm4);
            }
            float p[5];
            receiver_part(w, hp, p);
            own[0] = f4{p[0], p[1], p[2], p[3]};
            own[64] = gm16;
            own[128] = f4{p[4], gm4[0], gh[0], gh[1]};
            own[192] = f4{gh[2], 0, 0, 0};
            // the node's row for its senders, through LDS
            float* row = st + n * PG;
            *reinterpret_cast<f4*>(row + 4 * g) = f4{p[0], p[1], p[2], p[3]};
            *reinterpret_cast<f4*>(row + 16 + 4 * g) = gm16;
            row[32 + g] = p[4];
            row[36 + g] = gm4[0];
            lds_done();
            f4* to = reinterpret_cast<f4*>(a.pg[b & 1] + t * (VT_TILE * PG));
            const f4* from = reinterpret_cast<const f4*>(st);
            const f4 s0 = from[lane], s1 = from[64 + lane], s2 = from[128 + (lane & 31)];
            to[lane] = s0;
            to[64 + lane] = s1;
            if (lane < 32) to[128 + lane] = s2;
            lds_done();
            // weight gradients
            const float fov[3] = {fo[0], fo[1], fo[2]}, fiv[3] = {fi[0], fi[1], fi[2]};
            const float gfov[3] = {gfo[0], gfo[1], gfo[2]}, gfiv[3] = {gfi[0], gfi[1], gfi[2]};
            put_comps(st, 0, n, g, gz);
            put_comps(st, 10, n, g, hp);
            put_comps(st, 20, n, g, fov);
            put_comps(st, 30, n, g, fiv);
            put_comps(st, 40, n, g, gfov);
            put_comps(st, 50, n, g, gfiv);
            put_units(st, 60, n, g, m);
            put_comps(st, 80, n, g, gps);
            put_comps(st, 90, n, g, up);
            put_comps(st, 100, n, g, gzd);
            put_comps(st, 110, n, g, hc);
            if (g == 0) {
                st[120 * SR + n] = in.x;
                st[121 * SR + n] = in.y;
            }
            lds_done();
            const bool ten = n < 10;
            auto left = [&](int at) { return ten ? staged(st, at + n, g) : zero; };
            const f4 lz = left(0);
            // [h, c, 1, fo 0-3] and [fo 4-9, fi]
            product(3, lz, n < 11 ? staged(st, ten ? 10 + n : 120, g) : n == 11 ? one : staged(st, 8 + n, g));
            product(4, lz, staged(st, 24 + n, g));
            product(5, left(40), n < 11 ? staged(st, ten ? 60 + n : 121, g) : zero);
            product(6, left(50), n < 11 ? staged(st, ten ? 70 + n : 121, g) : zero);
            product(7, left(80), ten ? staged(st, 90 + n, g) : n == 10 ? one : zero);
            product(8, left(100), ten ? staged(st, 110 + n, g) : n == 10 ? one : zero);
            lds_done();
        }
    }
    // Sum of the wavefronts' accumulators: halves onto halves, through LDS.
    __syncthreads();
    float* const all = &pool[0][0];
    for (int half = EW / 2; half >= 1; half /= 2) {
        if (wave >= half && wave < 2 * half) {
            float* to = all + (wave - half) * (N_ACC * 64) + lane;
#pragma unroll
            for (int i = 0; i < N_ACC; ++i) to[i * 64] = acc[i];
        }
        __syncthreads();
        if (wave < half) {
            const float* from = all + wave * (N_ACC * 64) + lane;
#pragma unroll
            for (int i = 0; i < N_ACC; ++i) acc[i] += from[i * 64];
        }
        __syncthreads();
    }
    if (wave == 0) {
        float* to = a.part + ((size_t)(a.kbar - 1 - b) * gridDim.x + blockIdx.x) * (N_ACC * 64) + lane;
#pragma unroll
        for (int i = 0; i < N_ACC; ++i) to[i * 64] = acc[i];
    }
}
static_assert(EW / 2 * N_ACC * 64 <= EW * POOL, "accumulators of half the wavefronts fit the buffers");

// Accumulators of every backward launch summed over its workgroups, in order; added to
// the sums of the samples before (add).
__global__ __launch_bounds__(256) void train_gather_kernel(const float* __restrict__ part, int n_wg, int add,
                                                          double* __restrict__ red) {
    const int e = blockIdx.x * 256 + threadIdx.x;  // N_ACC * 64 is a multiple of 256
    const size_t at = (size_t)blockIdx.y * (N_ACC * 64) + e;
    const float* p = part + (size_t)blockIdx.y * n_wg * (N_ACC * 64) + e;
    double acc = add ? red[at] : 0.0;
#pragma unroll 8
    for (int i = 0; i < n_wg; ++i) acc += (double)p[(size_t)i * (N_ACC * 64)];
    red[at] = acc;
}
static_assert(N_ACC * 64 % 256 == 0, "whole workgroups");

// grad = scale * the accumulator entries of each weight (16 lanes of a per-lane sum).
__global__ __launch_bounds__(256) void train_scatter_kernel(const double* __restrict__ red,
                                                           const TrainEntry* __restrict__ ent, int kbar, double scale,
                                                           float* __restrict__ grad) {
    const int e = blockIdx.x * 256 + threadIdx.x, b = blockIdx.y;
    if (e >= TRAIN_NWB) return;
    const TrainEntry x = ent[e];
    const double* p = red + (size_t)(kbar - 1 - b + x.edges) * (N_ACC * 64) + x.at;
    double acc = 0.0;
    for (int i = 0; i < x.lanes; ++i) acc += p[i];
    grad[(size_t)b * TRAIN_NWB + e] = (float)(scale * (x.negative ? -acc : acc));
}

// Edge records of the tiles: in-edges of each node as the forward kernels order them,
// and the edges it sends.
__global__ __launch_bounds__(256) void train_edges_kernel(TrainEdgeArgs a) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int t = i / VT_TILE, n = i % VT_TILE;
    if (t >= a.n_tiles) return;
    const VtTile f = a.info[t];
    const int2 out = a.out_rows[t];
    const int slot = a.node[i].x;
    const size_t base = (size_t)f.x;
    // d = x_send - x_recv from the FP64 coordinates
    auto edge = [&](int recv, int send, int e) {
        TrainEdge v;
        v.dx = (float)(a.xy64[2 * (base + send)] - a.xy64[2 * (base + recv)]);
        v.dy = (float)(a.xy64[2 * (base + send) + 1] - a.xy64[2 * (base + recv) + 1]);
        v.nd = a.edge_nd[e];
        return v;
    };
    const TrainEdge none{-1, 0.0f, 0.0f, 0.0f};
    const int j = slot >= 0 ? slot - f.x : 0;
    const int e0 = slot >= 0 ? a.edge_ptr[slot] : 0, e1 = slot >= 0 ? a.edge_ptr[slot + 1] : 0;
    for (int s = 0; s < f.w; ++s) {
        TrainEdge v = none;
        if (e0 + s < e1) {
            const int l = a.edge_src[e0 + s];
            v = edge(j, l, e0 + s);
            v.node = a.pos[base + l];
        }
        a.rin[(size_t)(f.z + s) * VT_TILE + n] = v;
    }
    const int o0 = slot >= 0 ? a.oe_ptr[slot] : 0, o1 = slot >= 0 ? a.oe_ptr[slot + 1] : 0;
    for (int s = 0; s < out.y; ++s) {
        TrainEdge v = none;
        if (o0 + s < o1) {
            const int r = a.oe_recv[o0 + s];
            v = edge(r, j, a.oe_edge[o0 + s]);
            v.node = a.pos[base + r];
        }
        a.rout[(size_t)(out.x + s) * VT_TILE + n] = v;
    }
}

// Sum of squares of grad (one workgroup, fixed order) and the sum of the squared residuals.
__global__ __launch_bounds__(TB) void train_norm_kernel(const float* grad, int64_t nth, const double* sse, int n,
                                                       double* out) {
    __shared__ double red[TB / 64];
    double v = 0.0;
    for (int64_t e = threadIdx.x; e < nth; e += TB) v += (double)grad[e] * (double)grad[e];
    const double g2 = block_sum_d(v, red);
    double l = 0.0;
    for (int i = threadIdx.x; i < n; i += TB) l += sse[i];
    l = block_sum_d(l, red);
    if (threadIdx.x == 0) {
        out[0] = g2;
        out[1] = l;
    }
}

__global__ void adam_kernel(float* theta, const float* grad, float* m, float* v, int64_t n, float gscale, float lr,
                            float b1, float b2, float bc1, float bc2, float eps) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g = grad[i] * gscale;
    const float mi = b1 * m[i] + (1.0f - b1) * g;
    const float vi = b2 * v[i] + (1.0f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    theta[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
}

// r = b - A u into r (FP64), one row per thread.
__global__ void train_resid_kernel(const int32_t* rowptr, const int32_t* col, const double* val, const double* bb,
                                   const double* u, double* r, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double acc = 0.0;
    for (int q = rowptr[i]; q < rowptr[i + 1]; ++q) acc = fma(val[q], u[col[q]], acc);
    r[i] = bb[i] - acc;
}

// c_i = R_i r / |R_i r| per sub-mesh (0 where R_i r = 0), in slot order.
__global__ __launch_bounds__(TB) void train_rhs_kernel(const int32_t* sub_ptr, const int32_t* sub_nodes,
                                                       const double* r, float* c) {
    __shared__ double red[TB / 64];
    __shared__ double inv;
    const int sub = blockIdx.x;
    const int b = sub_ptr[sub], k = sub_ptr[sub + 1] - b;
    double v = 0.0;
    for (int j = threadIdx.x; j < k; j += TB) {
        const double x = r[sub_nodes[b + j]];
        v = fma(x, x, v);
    }
    const double ss = block_sum_d(v, red);
    if (threadIdx.x == 0) inv = ss > 0.0 ? 1.0 / sqrt(ss) : 0.0;
    __syncthreads();
    for (int j = threadIdx.x; j < k; j += TB) c[b + j] = (float)(r[sub_nodes[b + j]] * inv);
}

}  // namespace

// Positions of the weights (+ 1, signed; 0: zero) in a block's training blob, and of
// every weight's gradient in the accumulators.
void build_train_maps(std::vector<int32_t>& map, std::vector<TrainEntry>& ent) {
    auto phi1 = [](int u, int i) { return (u < D ? 0 : O_PI) + u % D * F_PHI + i; };
    auto phi1b = [](int u) { return (u < D ? 0 : O_PI) + D * F_PHI + u % D; };
    auto phi2 = [](int u, int o) { return (u < D ? 0 : O_PI) + D * F_PHI + D + o * D + u % D; };
    auto psi1 = [](int u, int i) { return O_PS + u * F_PSI + i; };
    auto psi2 = [](int o, int u) { return O_PS + D * F_PSI + D + o * D + u; };
    auto dec1 = [](int u, int i) { return O_DE + u * D + i; };
    const int dec2 = O_DE + D * D + D;
    // the forward blobs, built of positions instead of weights
    std::vector<float> pos((size_t)TRAIN_NWB), main, sender, dec;
    for (int i = 0; i < TRAIN_NWB; ++i) pos[i] = (float)(i + 1);
    build_vt_maps(pos.data(), main, sender, dec);
    map.assign((size_t)BLOB, 0);
    auto copy = [&](const std::vector<float>& v, int at) {
        for (size_t i = 0; i < v.size(); ++i) map[at + i] = (int32_t)v[i];
    };
    copy(main, 0);
    copy(sender, AT_SENDER);
    copy(dec, AT_DEC);
    auto put = [&](int at, int idx, int lane, int v) { map[at + (idx / 4 * 64 + lane) * 4 + idx % 4] = v + 1; };
    // operand of 16 rows: lane l holds row l % 16 (register i % 4 of group i / 4), input of group l / 16
    auto rows = [&](int at, int idx, auto f) {
        for (int l = 0; l < 64; ++l) put(at, idx, l, f(l % 16 % 4, l % 16 / 4, l / 16));
    };
    auto comps = [&](int at, int idx, int s, auto f) {  // rows and inputs are latent components
        rows(at, idx, [&](int r, int g, int kg) {
            const int i = r < 3 ? comp(g, r) : -1, u = comp(kg, s);
            return i < 0 || u < 0 ? -1 : f(i, u);
        });
    };
    for (int s = 0; s < 3; ++s) {
        for (int l = 0; l < 64; ++l)
            if (comp(l / 16, s) >= 0) put(AT_BACK, B_DV + s, l, dec2 + comp(l / 16, s));
        comps(AT_BACK, B_DT + s, s, [&](int i, int u) { return dec1(u, i); });
        comps(AT_BACK, B_P2 + s, s, [&](int i, int u) { return psi2(u, i); });
        comps(AT_BACK, B_GH + s, s, [&](int i, int u) { return psi1(u, i); });
        comps(AT_BACK, B_GO + s, s, [&](int i, int u) { return psi1(u, D + 1 + i); });
        comps(AT_BACK, B_GI + s, s, [&](int i, int u) { return psi1(u, 2 * D + 1 + i); });
        for (int in = 0; in < 2; ++in) {
            auto second = [&](int q, int kg) {  // unit q against message component kg feeds
                return q < 0 || comp(kg, s) < 0 || (q >= D) != (in == 1) ? -1 : phi2(q, comp(kg, s));
            };
            rows(AT_BACK, B_M16 + 3 * in + s, [&](int r, int g, int kg) { return second(unit(g, r), kg); });
            rows(AT_BACK, B_M4 + 3 * in + s, [&](int r, int g, int kg) { return second(r == 0 ? unit(g, 4) : -1, kg); });
        }
    }
    for (int r = 0; r < 5; ++r) {
        for (int l = 0; l < 64; ++l) {
            put(AT_EDGE, E_WX + r, l, phi1(unit(l / 16, r), 2 * D));
            put(AT_EDGE, E_WY + r, l, phi1(unit(l / 16, r), 2 * D + 1));
            put(AT_EDGE, E_WN + r, l, phi1(unit(l / 16, r), 2 * D + 2));
        }
        for (int side = 0; side < 2; ++side)
            rows(AT_EDGE, (side ? E_T2 : E_T1) + r, [&](int q, int g, int kg) {
                const int i = q < 3 ? comp(g, q) : -1;
                return i < 0 ? -1 : phi1(unit(kg, r), side * D + i);
            });
    }
    // gradients
    ent.assign((size_t)TRAIN_NWB, TrainEntry{});
    auto at = [&](int e, int prod, int row, int col, bool edges) {  // row: register row % 4 of group row / 4
        ent[e] = TrainEntry{(4 * prod + row % 4) * 64 + row / 4 * 16 + col, 1, (int8_t)edges, 0};
    };
    auto lanes = [&](int e, int acc, int g, bool edges, bool negative) {
        ent[e] = TrainEntry{acc * 64 + g * 16, 16, (int8_t)edges, (int8_t)negative};
    };
    for (int u = 0; u < 2 * D; ++u) {
        for (int i = 0; i < D; ++i) {
            at(phi1(u, i), u / 16, u % 16, i, true);
            at(phi1(u, D + i), (20 + u) / 16, (20 + u) % 16, i, true);
        }
        at(phi1b(u), u / 16, u % 16, 10, true);
        const int base = u < D ? 0 : O_PI;
        for (int o = 0; o < D; ++o) at(phi2(u, o), u < D ? 5 : 6, o, u % D, false);
        at(base + D * F_PHI + D + D * D + u % D, u < D ? 5 : 6, u % D, 10, false);
    }
    for (int g = 0; g < 4; ++g)
        for (int r = 0; r < 5; ++r) {
            const int u = unit(g, r);
            lanes(phi1(u, 2 * D), A_DX + r, g, true, u >= D);  // Phi_in sees -d
            lanes(phi1(u, 2 * D + 1), A_DY + r, g, true, u >= D);
            lanes(phi1(u, 2 * D + 2), A_N + r, g, true, false);
        }
    for (int u = 0; u < D; ++u) {
        for (int i = 0; i < D; ++i) {
            at(psi1(u, i), 3, u, i, false);
            at(psi1(u, D + 1 + i), i < 4 ? 3 : 4, u, i < 4 ? 12 + i : i - 4, false);
            at(psi1(u, 2 * D + 1 + i), 4, u, 6 + i, false);
            at(psi2(u, i), 7, u, i, false);
            at(dec1(u, i), 8, u, i, false);
        }
        at(psi1(u, D), 3, u, 10, false);
        at(O_PS + D * F_PSI + u, 3, u, 11, false);
        at(O_PS + D * F_PSI + D + D * D + u, 7, u, 10, false);
        at(O_DE + D * D + u, 8, u, 10, false);
    }
    for (int g = 0; g < 4; ++g)
        for (int r = 0; r < 3; ++r)
            if (comp(g, r) >= 0) lanes(dec2 + comp(g, r), A_UD + r, g, false, false);
    lanes(dec2 + D, A_GR, 0, false, false);
}

int64_t train_sse_count(int64_t tiles, int ks) { return (tiles * VT_TILE * ks + TB - 1) / TB; }

int train_workgroups(int64_t tiles) {
    const int64_t g = std::min<int64_t>((tiles + EW - 1) / EW, N_CU);
    return (int)((g + N_XCD - 1) / N_XCD * N_XCD);
}

hipError_t launch_train_edges(const TrainEdgeArgs& a, hipStream_t s) {
    if (a.n_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(train_edges_kernel, dim3((unsigned)(((int64_t)a.n_tiles * VT_TILE + 255) / 256)), dim3(256), 0, s,
                       a);
    return hipGetLastError();
}

hipError_t launch_train_grad(const TrainArgs& a, const float* theta, const int32_t* map, double* red, bool add,
                             hipStream_t s) {
    const int kb = a.kbar;
    const int64_t lanes = (int64_t)a.n_tiles * VT_TILE;
    const int64_t init = std::max<int64_t>(lanes, std::max(kb * ROW, 2 * PG));
    hipLaunchKernelGGL(train_blob_kernel, dim3((BLOB + 255) / 256, kb), dim3(256), 0, s, theta, map, a.blobs_out);
    hipLaunchKernelGGL(train_init_kernel, dim3((unsigned)((init + 255) / 256)), dim3(256), 0, s, a);
    // two workgroups per compute unit (LDS)
    const int64_t need = (a.n_tiles + EW - 1) / EW;
    const unsigned fg = (unsigned)((std::min<int64_t>(need, 2 * N_CU) + N_XCD - 1) / N_XCD * N_XCD);
    for (int b = 0; b + 1 < kb; ++b)
        hipLaunchKernelGGL(train_forward_kernel<false>, dim3(fg), dim3(EB), 0, s, a, b);
    hipLaunchKernelGGL(train_forward_kernel<true>, dim3(fg), dim3(EB), 0, s, a, kb - 1);
    const unsigned rg = (unsigned)train_sse_count(a.n_tiles, a.ks);
    hipLaunchKernelGGL(train_residual_kernel<true>, dim3(rg), dim3(TB), 0, s, a, a.r, a.rho);
    hipLaunchKernelGGL(train_residual_kernel<false>, dim3(rg), dim3(TB), 0, s, a, a.rho, a.gr);
    const unsigned bg = (unsigned)train_workgroups(a.n_tiles);
    hipLaunchKernelGGL((train_backward_kernel<false, true>), dim3(bg), dim3(EB), 0, s, a, kb - 1);
    for (int b = kb - 2; b >= 0; --b)
        hipLaunchKernelGGL((train_backward_kernel<true, true>), dim3(bg), dim3(EB), 0, s, a, b);
    hipLaunchKernelGGL((train_backward_kernel<true, false>), dim3(bg), dim3(EB), 0, s, a, -1);
    hipLaunchKernelGGL(train_gather_kernel, dim3(N_ACC * 64 / 256, kb + 1), dim3(256), 0, s, a.part, (int)bg, add ? 1 : 0,
                       red);
    return hipGetLastError();
}

hipError_t launch_train_reduce(const double* red, const TrainEntry* ent, int kbar, double scale, float* grad,
                               double* out2, const double* sse, int n_sse, hipStream_t s) {
    const int64_t nth = (int64_t)kbar * TRAIN_NWB;
    hipLaunchKernelGGL(train_scatter_kernel, dim3((TRAIN_NWB + 255) / 256, kbar), dim3(256), 0, s, red, ent, kbar,
                       scale, grad);
    hipLaunchKernelGGL(train_norm_kernel, dim3(1), dim3(TB), 0, s, grad, nth, sse, n_sse, out2);
    return hipGetLastError();
}

hipError_t launch_adam(float* theta, const float* grad, float* m, float* v, int64_t n, float gscale, float lr,
                       float b1, float b2, float bc1, float bc2, float eps, hipStream_t s) {
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, theta, grad, m, v, n, gscale,
                       lr, b1, b2, bc1, bc2, eps);
    return hipGetLastError();
}

hipError_t launch_train_rhs(const int32_t* rowptr, const int32_t* col, const double* val, const double* bb,
                            const double* u, double* r, int n, const int32_t* sub_ptr, const int32_t* sub_nodes,
                            int K, float* c, hipStream_t s) {
    hipLaunchKernelGGL(train_resid_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, rowptr, col, val, bb,
                       u, r, n);
    hipLaunchKernelGGL(train_rhs_kernel, dim3((unsigned)K), dim3(TB), 0, s, sub_ptr, sub_nodes, r, c);
    return hipGetLastError();
}

}  // namespace ddmgnn
