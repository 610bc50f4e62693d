// FP64 and FP32 DSS_theta forward (Sec. III.B, eqs. (14)-(18)) of width 10 on
// matrix cores, one launch per message-passing block.
//
// Why a launch per block: one workgroup per sub-mesh leaves the chip idle when
// there are few sub-meshes and waits for the largest one when there are not many
// more than compute units. Here the units of work are tiles of 16 nodes, spread
// over all compute units whatever the sub-meshes' sizes; the price is a launch
// per block (1.7 us inside a captured graph) and the latent state and sender rows
// in device memory. One forward of 30 blocks, one workgroup per sub-mesh before
// and tiles now: 5k nodes in 8 parts, FP64 829 -> 168 us, FP32 421 -> 137; 100k
// in 150, FP64 2,060 -> 563, FP32 580 -> 419; 1M in 1500, FP64 11.2 -> 6.2 ms.
//
// A wavefront takes a tile: lane l serves node l % 16 and group l / 16. The
// twenty hidden units of the two message layers are spread over the groups,
// five per lane (unit()), so the edge loop needs no cross-lane step and its
// sums are the next layer's matrix operand as they lie: v_mfma_*_16x16x4 takes
// operand entry k from group k, and the rows of the weight operands are
// permuted on the host so that every result lands where the next layer reads
// it. Both instructions accumulate as a chain of fused multiply-adds in
// ascending k (checked on the device), so each FP32 value is the one of a
// scalar loop over the inputs in order: the FP32 results equal those of the
// vector kernel they replaced, bit for bit. In FP64 the second message layers
// are folded into Psi's hidden layer (no activation lies between them), the
// centred coordinates are two more inputs of the first layer, and c and the
// in-degree two more of Psi's.
//
// Sender rows Q (20 values per slot, five per group) alternate between two
// buffers: block k reads one while it writes block k + 1's into the other.
#include <hip/hip_runtime.h>

#include "ddmgnn.h"
#include "dss_tile.h"
#include "setup.h"
#include "tile.h"

namespace ddmgnn {

namespace {

template <typename T>
__device__ __forceinline__ const VtVecs<T>& vecs(const DevProb& P);
template <>
__device__ __forceinline__ const VtVecs<double>& vecs<double>(const DevProb& P) { return P.vt64; }
template <>
__device__ __forceinline__ const VtVecs<float>& vecs<float>(const DevProb& P) { return P.vt32; }

// Sender rows of tile t's nodes from their latent state (h; FP64: the coordinates
// are h's last two entries) into Q, through the wavefront's buffer buf.
template <typename T>
__device__ __forceinline__ void sender_rows(const T* blob, int lane, const T (&h)[3], T x, T y, size_t t, T* buf,
                                            T* __restrict__ Q) {
    using L = VtLayout<T>;
    const int n = lane & 15, g = lane >> 4;
    typename Mx<T>::A4 acc = {0, 0, 0, 0};
    T q[5];
    const WeightBlob<T, L::N_Q, L::N_QOPS> w{blob, lane};
    if constexpr (sizeof(T) == 8) {
        T q4 = 0;
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            acc = Mx<T>::mm(w[L::Q16 + s], h[s], acc);
            q4 = __builtin_amdgcn_mfma_f64_4x4x4f64(w[L::Q4 + s], h[s], q4, 0, 0, 0);
        }
        q[4] = q4;
    } else {
        // coordinate part first, then the chain over h (Phi_in sees -d)
        T c[5];
#pragma unroll
        for (int r = 0; r < 5; ++r) c[r] = fma(w[L::QX + r], x, w[L::QY + r] * y);
        acc[0] = c[0];
        acc[1] = c[1];
        acc[2] = -c[2];
        acc[3] = -c[3];
        typename Mx<T>::A4 acc4 = {g < 2 ? c[4] : -c[4], 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            acc = Mx<T>::mm(w[L::Q16 + s], h[s], acc);
            acc4 = Mx<T>::mm(w[L::Q4 + s], h[s], acc4);
        }
        q[4] = acc4[0];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) q[r] = acc[r];
    using C = typename Mx<T>::Chunk;
    row_put<T>(buf + n * ROW, g, q);
    lds_done();
    C* to = reinterpret_cast<C*>(Q + t * (VT_TILE * ROW));
    constexpr int P = VT_TILE * Rows20<T>::PIECES;  // 80 or 160
#pragma unroll
    for (int i = 0; i < P; i += 64)
        if (i + lane < P) to[i + lane] = reinterpret_cast<const C*>(buf)[i + lane];
    lds_done();
}

// Sums as the single-workgroup kernels form them: over 1024 virtual threads
// (node j belongs to thread j % 1024), a shuffle tree per wavefront, then the
// wavefronts in order.
constexpr int RB = 1024;
__device__ inline double restrict_sum(double v, double* sh) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double acc = 0.0;
    for (int i = 0; i < RB / 64; ++i) acc += sh[i];
    return acc;
}

// s_i = |R_i r|, y0_i = (R_0 r)_i, c_i = R_i r / s_i (or the given c), the zero
// latent state and the sender rows of block 0. One workgroup per sub-mesh.
template <typename T>
__global__ __launch_bounds__(RB) void dss_restrict_kernel(const DevProb* __restrict__ tab,
                                                         const int2* __restrict__ work, const T* __restrict__ qblob,
                                                         int apply) {
    const int2 wi = work[blockIdx.x];
    const DevProb& P = tab[wi.x];
    if (P.st && P.st->done) return;
    __shared__ double cj[kMaxSubNodes];
    __shared__ double red[RB / 64];
    __shared__ __align__(16) T sw[VtBlobs<T>::Q];
    __shared__ __align__(16) T buf[RB / 64][VT_TILE * ROW];
    stage<T, VtBlobs<T>::Q / 64, RB>(qblob, sw);
    const int sub = wi.y, tid = threadIdx.x;
    const int base = P.sub_ptr[sub], k = P.sub_ptr[sub + 1] - base;
    if (apply) {
        const double* __restrict__ r = P.r;
        double ss = 0.0, yy = 0.0;
        for (int j = tid; j < k; j += RB) {
            const double v = r[P.sub_nodes[base + j]];
            cj[j] = v;
            ss = fma(v, v, ss);
            yy = fma(P.weights[base + j], v, yy);
        }
        ss = restrict_sum(ss, red);
        yy = restrict_sum(yy, red);
        const double sn = sqrt(ss);
        if (tid == 0) {
            P.s[sub] = sn;
            P.y0[sub] = yy;
        }
        // R_i r = 0: c = 0, and the last block writes a zero local term
        for (int j = tid; j < k; j += RB) cj[j] = sn == 0.0 ? 0.0 : cj[j] / sn;
    } else {
        for (int j = tid; j < k; j += RB) cj[j] = P.c_in[base + j];
    }
    vmem_done();
    __syncthreads();
    const VtVecs<T>& V = vecs<T>(P);
    const int lane = tid & 63, n = lane & 15, g = lane >> 4;
    const int t0 = P.vt_first[sub], t1 = t0 + (k + VT_TILE - 1) / VT_TILE;
    for (int t = t0 + (tid >> 6); t < t1; t += RB / 64) {
        const int2 nd = P.vt_node[(size_t)t * VT_TILE + n];
        const size_t sl = nd.x >= 0 ? (size_t)nd.x : (size_t)base;
        const T c = nd.x >= 0 ? (T)cj[nd.x - base] : (T)0;
        T x, y, h[3] = {0, 0, 0};
        if constexpr (sizeof(T) == 8) {  // coordinates relative to the sub-mesh's first node
            x = P.xy64[2 * sl] - P.xy64[2 * (size_t)base];
            y = P.xy64[2 * sl + 1] - P.xy64[2 * (size_t)base + 1];
            if (g >= 2) h[2] = g == 2 ? x : y;
        } else {
            x = P.xyc32[2 * sl];
            y = P.xyc32[2 * sl + 1];
            if (g == 0) reinterpret_cast<f4*>(V.info)[(size_t)t * VT_TILE + n] = f4{x, y, (T)nd.y, c};
        }
        store_h<T>(V.h, (size_t)t, lane, h, g == 2 ? c : (T)nd.y);
        sender_rows<T>(sw, lane, h, x, y, (size_t)t, buf[tid >> 6], V.q[0]);
    }
}

template <typename T>
struct VtArgs {
    const DevProb* tab;
    const int4* tiles;
    int n_tiles;
    int solo;
    int apply;
    int from;        // sender buffer read by this block
    T alpha;
    const T* main;   // this block's blob
    const T* next;   // the next block's sender blob, or (last block) the decoder's
};

// One message-passing block of every tile; the last one decodes instead of
// writing the next sender rows. With few tiles the time is the chain of
// dependent loads (tile -> edge records -> sender rows) and matrix products of
// one tile, about 3 us; with many, the wavefronts in flight over that chain, and
// from about 50,000 tiles (FP32; half that in FP64) HBM: 440 MB per FP32 block of
// 85,000 tiles in 115 us. So few, wide loads (each costs 16 cycles of the address
// unit whatever its width): edge records and sender rows go straight to LDS, a
// tile's state and inputs are one or two loads, and the next tile's are issued
// before Psi. The weights lie in LDS, shared by the workgroup (in registers they
// would halve the wavefronts in flight). The tiles are dealt to the eight dies in
// contiguous slabs, so that a sub-mesh's sender rows are gathered through one
// die's L2.
//
// Workgroups of a wavefront per SIMD, so that they spread evenly, as many as the LDS holds
// (FP64: 40,960 bytes each; the last block's, with the decoder's weights, three). 100k nodes in 150
// parts, one forward: FP32 419 us, FP64 563; two of eight wavefronts 439 and 584. More than 16
// wavefronts per compute unit are slower (FP32, 22: 467).
constexpr int BLOCK = 256, WG_PER_CU = 4;
template <typename T, bool LAST>
__global__ __launch_bounds__(BLOCK, LAST && sizeof(T) == 8 ? WG_PER_CU - 1 : WG_PER_CU) void dss_block_kernel(VtArgs<T> a) {
    using L = VtLayout<T>;
    using M = Mx<T>;
    using A4 = typename M::A4;
    using R = Rows20<T>;
    constexpr size_t MAIN = VtBlobs<T>::MAIN, NEXT = LAST ? VtBlobs<T>::DEC : VtBlobs<T>::Q;
    __shared__ __align__(16) T sw[MAIN];
    __shared__ __align__(16) T swn[NEXT];
    __shared__ __align__(16) T buf[BLOCK / 64][R::BUF];
    __shared__ __align__(16) VtRec<T> recs[BLOCK / 64][R::RECS];
    const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int die = blockIdx.x % N_XCD;
    const int nw = (int)(gridDim.x / N_XCD) * (BLOCK / 64);
    const int end = (int)((int64_t)a.n_tiles * (die + 1) / N_XCD);
    int it = (int)((int64_t)a.n_tiles * die / N_XCD) + (int)(blockIdx.x / N_XCD) * (BLOCK / 64) + wave;
    auto done = [](const DevProb* p) {
        const KState* st = uload(&p->st);
        return st && uload(&st->done);
    };
    if (a.solo && done(a.tab)) return;
    stage<T, MAIN / 64, BLOCK>(a.main, sw);
    stage<T, NEXT / 64, BLOCK>(a.next, swn);
    // Pieces this lane gathers of a chunk's rows: the (edge row, node) and the byte offset in the row.
    int gat[R::LOADS], off[R::LOADS];
#pragma unroll
    for (int i = 0; i < R::LOADS; ++i) {
        gat[i] = (i * 64 + lane) / R::PIECES;
        off[i] = (i * 64 + lane) % R::PIECES * 16;
    }
    auto read_recs = [&](const VtRec<T>* from) {  // VT_ROWS edge rows
#pragma unroll
        for (int i = 0; i < R::RECS * (int)sizeof(VtRec<T>) / 1024; ++i)
            to_lds(reinterpret_cast<const char*>(from) + i * 1024 + lane * 16,
                   reinterpret_cast<char*>(recs[wave]) + i * 1024);
    };
    // The next tile whose problem still runs (it = end: none), and the loads of what
    // a lane needs of it before its sender rows: edge records (LDS), state and inputs.
    const DevProb* P = a.tab;
    i4 wi = {0, 0, 0, 0};
    T hn[3], x4n = 0;
    f4 infon = {0, 0, 0, 0};
    auto fetch = [&]() {
        for (; it < end; it += nw) {
            wi = uload(reinterpret_cast<const i4*>(a.tiles) + it);
            if (a.solo) break;
            P = a.tab + wi[0];
            if (!done(P)) break;
        }
        if (it >= end) return;
        const VtVecs<T>& V = vecs<T>(*P);
        read_recs(uload(&V.rec) + (size_t)wi[2] * VT_TILE);
        load_h<T>(uload(&V.h), (size_t)wi[1], lane, hn, x4n);
        if constexpr (sizeof(T) == 4)
            infon = reinterpret_cast<const f4*>(uload(&V.info))[(size_t)wi[1] * VT_TILE + n];
    };
    fetch();
    vmem_done();
    __syncthreads();
    const WeightBlob<T, L::N_MAIN, L::N_OPS> w{sw, lane};
    const LaneBlob<T> wn{swn, lane};  // the decoder's
    while (it < end) {
        asm volatile("" ::: "memory");  // keeps the weights in LDS: hoisted, they would fill the registers
        const DevProb* PA = P;
        const size_t t = (size_t)wi[1];
        const int md = wi[3];
        const VtVecs<T>& V = vecs<T>(*P);
        const VtRec<T>* rec = uload(&V.rec) + (size_t)wi[2] * VT_TILE;
        const char* __restrict__ Q = reinterpret_cast<const char*>(uload(&V.q[a.from]));
        T* const hout = uload(&V.h);
        T* const qout = uload(&V.q[a.from ^ 1]);
        vmem_done();
        T h[3] = {hn[0], hn[1], hn[2]};
        const T x4 = x4n;
        const f4 info = infon;
        T x = 0, y = 0;
        if constexpr (sizeof(T) == 4) {
            x = info[0];
            y = info[1];
        }

        // Receiver part of the first message layers.
        T p[5];
        {
            A4 acc = {w[L::CP], w[L::CP + 1], w[L::CP + 2], w[L::CP + 3]};
            if constexpr (sizeof(T) == 8) {
                T p4 = w[L::CP4];
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    acc = M::mm(w[L::P16 + s], h[s], acc);
                    p4 = __builtin_amdgcn_mfma_f64_4x4x4f64(w[L::P4 + s], h[s], p4, 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) p[r] = acc[r];
                p[4] = p4;
            } else {
                A4 acc4 = {w[L::CP4], 0, 0, 0};
#pragma unroll
                for (int s = 0; s < 3; ++s) {
                    acc = M::mm(w[L::P16 + s], h[s], acc);
                    acc4 = M::mm(w[L::P4 + s], h[s], acc4);
                }
                // minus W_d x (Phi_out), plus W_d x (Phi_in)
#pragma unroll
                for (int r = 0; r < 5; ++r) {
                    const T v = r < 4 ? acc[r < 4 ? r : 0] : acc4[0];
                    const T wx = w[L::WX + r], wy = w[L::WY + r];
                    const T po = v - fma(wx, x, wy * y);
                    const T pi = fma(wx, x, fma(wy, y, v));
                    p[r] = r < 2 ? po : r < 4 ? pi : g < 2 ? po : pi;
                }
            }
        }

        // Message sums over the in-edges, EDGES rows of senders at a time. Missing
        // edges read the sentinel row (-inf), whose message is max(-inf, 0) = 0.
        T m[5] = {0, 0, 0, 0, 0};
        for (int e0 = 0; e0 < md; e0 += VT_ROWS) {
            if (e0) {
                lds_done();
                read_recs(rec + e0 * VT_TILE);
                vmem_done();
            }
            for (int e = 0; e < VT_ROWS && e0 + e < md; e += R::EDGES) {
                int l[R::LOADS];
#pragma unroll
                for (int i = 0; i < R::LOADS; ++i) l[i] = recs[wave][e * VT_TILE + gat[i]].src;
                lds_done();  // also: the rows of the previous chunk have been read
#pragma unroll
                for (int i = 0; i < R::LOADS; ++i)
                    to_lds(Q + (size_t)l[i] * (ROW * sizeof(T)) + off[i], reinterpret_cast<char*>(buf[wave]) + i * 1024);
                T d[R::EDGES];
#pragma unroll
                for (int i = 0; i < R::EDGES; ++i) d[i] = recs[wave][(e + i) * VT_TILE + n].nd;
                vmem_done();
#pragma unroll
                for (int i = 0; i < R::EDGES; i += 2)
                    if (e0 + e + i < md) {  // uniform; md is even
                        T q[2][5];
#pragma unroll
                        for (int f = 0; f < 2; ++f) row_get<T>(buf[wave] + ((i + f) * VT_TILE + n) * ROW, g, q[f]);
#pragma unroll
                        for (int f = 0; f < 2; ++f)
#pragma unroll
                            for (int r = 0; r < 5; ++r) m[r] += M::relu(fma(w[L::WN + r], d[i + f], p[r] + q[f][r]));
                    }
            }
        }
        lds_done();
        it += nw;
        fetch();

        // Psi.
        A4 hid = {w[L::CH], w[L::CH + 1], w[L::CH + 2], 0};
        A4 out = {w[L::CO], w[L::CO + 1], w[L::CO + 2], 0};
        if constexpr (sizeof(T) == 8) {
            // ten rows: three products of four rows are 48 cycles, one of sixteen 64, and their
            // three chains hide each other's latency
            const QuadBlob w4{sw, lane};
            const T in[8] = {h[0], h[1], g >= 2 ? x4 : h[2], m[0], m[1], m[2], m[3], m[4]};
#pragma unroll
            for (int s = 0; s < 8; ++s)
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    hid[q] = __builtin_amdgcn_mfma_f64_4x4x4f64(w4[L::HID + 3 * s + q], in[s], hid[q], 0, 0, 0);
#pragma unroll
            for (int s = 0; s < 3; ++s)
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    out[q] = __builtin_amdgcn_mfma_f64_4x4x4f64(w4[L::OUT + 3 * s + q], M::relu(hid[s]), out[q], 0, 0, 0);
        } else {
            const T deg = info[2], c = info[3];
            // An operand's entries against zero weights are zeroed: an overflowed one would be
            // a NaN in the product, and relu drops NaN.
            const T m4o = g < 2 ? m[4] : (T)0, m4i = g < 2 ? (T)0 : m[4];
            A4 fo = {w[L::CCO] * deg, w[L::CCO + 1] * deg, w[L::CCO + 2] * deg, 0};
            A4 fi = {w[L::CCI] * deg, w[L::CCI + 1] * deg, w[L::CCI + 2] * deg, 0};
            fo = M::mm(w[L::FO], m[0], fo);
            fi = M::mm(w[L::FI], m[2], fi);
            fo = M::mm(w[L::FO + 1], m[1], fo);
            fi = M::mm(w[L::FI + 1], m[3], fi);
            fo = M::mm(w[L::FO + 2], m4o, fo);
            fi = M::mm(w[L::FI + 2], m4i, fi);
            fo[2] = g < 2 ? fo[2] : (T)0;
            fi[2] = g < 2 ? fi[2] : (T)0;
            hid = M::mm(w[L::HID], h[0], hid);
            hid = M::mm(w[L::HID + 1], h[1], hid);
            hid = M::mm(w[L::HID + 2], g == 2 ? c : h[2], hid);
#pragma unroll
            for (int s = 0; s < 3; ++s) hid = M::mm(w[L::HID + 3 + s], fo[s], hid);
#pragma unroll
            for (int s = 0; s < 3; ++s) hid = M::mm(w[L::HID + 6 + s], fi[s], hid);
#pragma unroll
            for (int s = 0; s < 3; ++s) out = M::mm(w[L::OUT + s], M::relu(hid[s]), out);
        }
        // entries past the last component stay: FP64 keeps its coordinates there, FP32 zeros
        // (their rows of the products are zero weights times values that may have overflowed)
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const T v = fma(a.alpha, out[r], h[r]);
            if (r < 2 || g < 2) h[r] = v;
        }

        if constexpr (!LAST) {
            store_h<T>(hout, t, lane, h, x4);
            sender_rows<T>(swn, lane, h, x, y, t, buf[wave], qout);
        } else {
            // Decoder: r~ = D(h).
            A4 dh = {wn[L::CDH], wn[L::CDH + 1], wn[L::CDH + 2], 0};
#pragma unroll
            for (int s = 0; s < 3; ++s) dh = M::mm(wn[L::DH + s], h[s], dh);
            A4 r = {wn[L::CDO], 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 3; ++s) r = M::mm(wn[L::DO + s], M::relu(dh[s]), r);
            const int slot = uload(&PA->vt_node)[t * VT_TILE + n].x;
            if (g == 0 && slot >= 0) {
                double z = (double)r[0];
                if (a.apply) {
                    const double sn = PA->s[PA->slot_sub[slot]];
                    z = sn == 0.0 ? 0.0 : sn * z;
                }
                PA->local[slot] = z;
            }
        }
    }
}

// Nodes of every tile lane, and the tile position of every slot.
__global__ __launch_bounds__(VT_BLOCK) void vt_nodes_kernel(const DevProb* __restrict__ tab,
                                                           const VtTile* __restrict__ info, int n_tiles,
                                                           int2* __restrict__ node, int32_t* __restrict__ pos) {
    const int i = blockIdx.x * VT_BLOCK + threadIdx.x;
    const int t = i / VT_TILE, n = i % VT_TILE;
    if (t >= n_tiles) return;
    const DevProb& P = *tab;
    const VtTile f = info[t];
    const int k = P.sub_ptr[P.slot_sub[f.x] + 1] - f.x;
    const bool in = f.y + n < k;
    const int slot = in ? f.x + P.tiles[f.x + f.y + n].j : -1;
    node[i] = make_int2(slot, in ? P.edge_ptr[slot + 1] - P.edge_ptr[slot] : 0);
    if (in) pos[slot] = i;
}

// Records of every edge row: the in-edges of each node in order, then sentinels.
template <typename T>
__global__ __launch_bounds__(VT_BLOCK) void vt_edges_kernel(const DevProb* __restrict__ tab,
                                                           const VtTile* __restrict__ info, int n_tiles,
                                                           const int2* __restrict__ node,
                                                           const int32_t* __restrict__ pos, VtRec<T>* __restrict__ rec) {
    const int i = blockIdx.x * VT_BLOCK + threadIdx.x;
    const int t = i / VT_TILE, n = i % VT_TILE;
    if (t >= n_tiles) return;
    const DevProb& P = *tab;
    const VtTile f = info[t];
    const int slot = node[i].x, deg = node[i].y;
    const size_t base = (size_t)f.x, sl = slot >= 0 ? (size_t)slot : base;
    const int e0 = P.edge_ptr[sl];
    for (int s = 0; s < f.w; ++s) {
        VtRec<T> v{};
        v.src = n_tiles * VT_TILE;
        if (s < deg) {
            const size_t l = base + P.edge_src[e0 + s];
            v.src = pos[l];
            if constexpr (sizeof(T) == 4) {
                v.nd = P.edge_nd[e0 + s];
            } else {
                const double dx = P.xy64[2 * l] - P.xy64[2 * sl], dy = P.xy64[2 * l + 1] - P.xy64[2 * sl + 1];
                v.nd = sqrt(dx * dx + dy * dy);
            }
        }
        rec[(size_t)(f.z + s) * VT_TILE + n] = v;
    }
}

template <typename T>
__global__ __launch_bounds__(VT_BLOCK) void vt_fill_kernel(T* __restrict__ p, int64_t n, T v) {
    const int64_t i = (int64_t)blockIdx.x * VT_BLOCK + threadIdx.x;
    if (i < n) p[i] = v;
}

template <typename T>
hipError_t fill(T* p, int64_t n, T v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(vt_fill_kernel<T>, dim3((unsigned)((n + VT_BLOCK - 1) / VT_BLOCK)), dim3(VT_BLOCK), 0, s, p, n,
                       v);
    return hipGetLastError();
}

// ------------------------------------------------------------------ weight blobs (host)
constexpr int IN_PHI = 2 * D + 3, IN_PSI = 3 * D + 1;
constexpr int OFF_PI = D * IN_PHI + D + D * D + D;
constexpr int OFF_PS = 2 * OFF_PI;
constexpr int OFF_DE = OFF_PS + D * IN_PSI + D + D * D + D;
constexpr int BLOCK_W = OFF_DE + D * D + D + D + 1;

// Weights of one block as double.
struct Wts {
    const float* w;
    double phi1(int u, int i) const { return w[(u < D ? 0 : OFF_PI) + (u % D) * IN_PHI + i]; }  // u: 0-19
    double phi1b(int u) const { return w[(u < D ? 0 : OFF_PI) + D * IN_PHI + u % D]; }
    double phi2(bool in, int o, int u) const { return w[(in ? OFF_PI : 0) + D * IN_PHI + D + o * D + u]; }
    double phi2b(bool in, int o) const { return w[(in ? OFF_PI : 0) + D * IN_PHI + D + D * D + o]; }
    double psi1(int u, int i) const { return w[OFF_PS + u * IN_PSI + i]; }
    double psi1b(int u) const { return w[OFF_PS + D * IN_PSI + u]; }
    double psi2(int o, int u) const { return w[OFF_PS + D * IN_PSI + D + o * D + u]; }
    double psi2b(int o) const { return w[OFF_PS + D * IN_PSI + D + D * D + o]; }
    double dec1(int u, int i) const { return w[OFF_DE + u * D + i]; }
    double dec1b(int u) const { return w[OFF_DE + D * D + u]; }
    double dec2(int u) const { return w[OFF_DE + D * D + D + u]; }
    double dec2b() const { return w[OFF_DE + D * D + 2 * D]; }
};

// Writes value idx of lane l of a blob.
template <typename T>
void put(T* blob, int idx, int lane, double v) {
    constexpr int PER = Mx<T>::PER;
    blob[((size_t)(idx / PER) * 64 + lane) * PER + idx % PER] = (T)v;
}

// Operand A of 16 rows: lane l holds row l % 16, input of group l / 16. f(r, g, kg):
// weight of the result register r of group g against the entry that group kg feeds.
template <typename T, class F>
void put_a16(T* blob, int idx, F f) {
    for (int l = 0; l < 64; ++l) {
        const int i = l % 16, kg = l / 16;
        const int r = sizeof(T) == 8 ? i / 4 : i % 4, g = sizeof(T) == 8 ? i % 4 : i / 4;
        put(blob, idx, l, f(r, g, kg));
    }
}
// Operand A of the 4-row FP64 product: lane l holds row l % 4 (= group), input of group l / 16.
template <class F>
void put_a4(double* blob, int idx, F f) {
    for (int l = 0; l < 64; ++l) put(blob, idx, l, f(l % 4, l / 16));
}
// Per-lane constant of result register r: f(r, g).
template <typename T, class F>
void put_c(T* blob, int idx, F f) {
    for (int l = 0; l < 64; ++l) put(blob, idx, l, f(l / 16));
}

// Weight of a first message layer's unit u against the latent component that group
// kg feeds in step s (off: 0 receiver, D sender); FP64: the coordinates follow in step 2.
template <typename T>
double first_layer(const Wts& w, int u, int s, int kg, int off) {
    const int i = comp(kg, s);
    if (i >= 0) return w.phi1(u, off + i);
    if (sizeof(T) == 4) return 0.0;
    // d = x_sender - x_receiver for Phi_out, its negative for Phi_in
    const double sign = ((u < D) == (off == D)) ? 1.0 : -1.0;
    return sign * w.phi1(u, 2 * D + (kg - 2));
}

template <typename T>
void build_first(const Wts& w, T* blob, int i16, int i4, int off) {
    for (int s = 0; s < 3; ++s) {
        put_a16(blob, i16 + s, [&](int r, int g, int kg) { return first_layer<T>(w, unit(g, r), s, kg, off); });
        if constexpr (sizeof(T) == 8)
            put_a4(blob, i4 + s, [&](int g, int kg) { return first_layer<T>(w, unit(g, 4), s, kg, off); });
        else
            put_a16(blob, i4 + s, [&](int r, int g, int kg) {
                return r == 0 ? first_layer<T>(w, unit(g, 4), s, kg, off) : 0.0;
            });
    }
}

template <typename T>
void build_main(const Wts& w, T* blob) {
    using L = VtLayout<T>;
    build_first<T>(w, blob, L::P16, L::P4, 0);
    for (int r = 0; r < 4; ++r) put_c(blob, L::CP + r, [&](int g) { return w.phi1b(unit(g, r)); });
    put_c(blob, L::CP4, [&](int g) { return w.phi1b(unit(g, 4)); });
    for (int r = 0; r < 5; ++r) put_c(blob, L::WN + r, [&](int g) { return w.phi1(unit(g, r), 2 * D + 2); });
    auto component = [&](int idx, auto f) {  // weights whose rows are latent components
        auto row = [&](int r, int g, int kg) {
            const int u = r < 3 ? comp(g, r) : -1;
            return u < 0 ? 0.0 : f(u, kg);
        };
        if constexpr (sizeof(T) == 8) {  // QuadBlob: the three operands of step idx
            for (int r = 0; r < 3; ++r)
                for (int l = 0; l < 16; ++l) {
                    const int i = 3 * idx + r;
                    blob[(i / 2 * 16 + l) * 2 + i % 2] = row(r, l % 4, l / 4);
                }
        } else {
            put_a16(blob, idx, row);
        }
    };
    auto constant = [&](int idx, auto f) {
        for (int r = 0; r < 3; ++r)
            put_c(blob, idx + r, [&](int g) { return comp(g, r) < 0 ? 0.0 : f(comp(g, r)); });
    };
    constant(L::CH, [&](int u) { return w.psi1b(u); });
    constant(L::CO, [&](int u) { return w.psi2b(u); });
    for (int s = 0; s < 3; ++s)
        component((sizeof(T) == 8 ? L::OUT / 3 : L::OUT) + s, [&](int o, int kg) { return comp(kg, s) < 0 ? 0.0 : w.psi2(o, comp(kg, s)); });
    // entries of the third h step past the components: c, and (FP64) the in-degree
    auto past = [&](int u, int kg) {
        if (kg == 2) return w.psi1(u, D);
        if (sizeof(T) == 4) return 0.0;
        double v = 0.0;
        for (int o = 0; o < D; ++o)
            v += w.psi1(u, D + 1 + o) * w.phi2b(false, o) + w.psi1(u, 2 * D + 1 + o) * w.phi2b(true, o);
        return v;
    };
    for (int s = 0; s < 3; ++s)
        component(L::HID + s, [&](int u, int kg) { return comp(kg, s) < 0 ? past(u, kg) : w.psi1(u, comp(kg, s)); });
    if constexpr (sizeof(T) == 8) {
        for (int s = 0; s < 5; ++s)
            component(L::HID + 3 + s, [&](int u, int kg) {  // Psi's weights times the second message layer's
                const int q = unit(kg, s);
                double v = 0.0;
                for (int o = 0; o < D; ++o) v += w.psi1(u, (q < D ? 1 : 2) * D + 1 + o) * w.phi2(q >= D, o, q % D);
                return v;
            });
    } else {
        for (int s = 0; s < 3; ++s) {
            // message sums of Phi_out lie in units 0, 1 and 4 of the lanes, of Phi_in in 2, 3 and 4
            component(L::FO + s, [&](int o, int kg) {
                const int q = unit(kg, s < 2 ? s : 4);
                return q < D ? w.phi2(false, o, q) : 0.0;
            });
            component(L::FI + s, [&](int o, int kg) {
                const int q = unit(kg, s < 2 ? 2 + s : 4);
                return q >= D ? w.phi2(true, o, q - D) : 0.0;
            });
            component(L::HID + 3 + s,
                      [&](int u, int kg) { return comp(kg, s) < 0 ? 0.0 : w.psi1(u, D + 1 + comp(kg, s)); });
            component(L::HID + 6 + s,
                      [&](int u, int kg) { return comp(kg, s) < 0 ? 0.0 : w.psi1(u, 2 * D + 1 + comp(kg, s)); });
        }
        constant(L::CCO, [&](int o) { return w.phi2b(false, o); });
        constant(L::CCI, [&](int o) { return w.phi2b(true, o); });
        for (int r = 0; r < 5; ++r) {
            put_c(blob, L::WX + r, [&](int g) { return w.phi1(unit(g, r), 2 * D); });
            put_c(blob, L::WY + r, [&](int g) { return w.phi1(unit(g, r), 2 * D + 1); });
        }
    }
}

template <typename T>
void build_sender(const Wts& w, T* blob) {
    using L = VtLayout<T>;
    build_first<T>(w, blob, L::Q16, L::Q4, D);
    if constexpr (sizeof(T) == 4)
        for (int r = 0; r < 5; ++r) {
            put_c(blob, L::QX + r, [&](int g) { return w.phi1(unit(g, r), 2 * D); });
            put_c(blob, L::QY + r, [&](int g) { return w.phi1(unit(g, r), 2 * D + 1); });
        }
}

template <typename T>
void build_dec(const Wts& w, T* blob) {
    using L = VtLayout<T>;
    for (int s = 0; s < 3; ++s) {
        put_a16(blob, L::DH + s, [&](int r, int g, int kg) {
            const int u = r < 3 ? comp(g, r) : -1;
            return u < 0 || comp(kg, s) < 0 ? 0.0 : w.dec1(u, comp(kg, s));
        });
        put_a16(blob, L::DO + s, [&](int r, int g, int kg) {
            return r == 0 && g == 0 && comp(kg, s) >= 0 ? w.dec2(comp(kg, s)) : 0.0;
        });
    }
    for (int r = 0; r < 3; ++r)
        put_c(blob, L::CDH + r, [&](int g) { return comp(g, r) < 0 ? 0.0 : w.dec1b(comp(g, r)); });
    put_c(blob, L::CDO, [&](int g) { return g == 0 ? w.dec2b() : 0.0; });
}

// A blob of N values per lane in the form of the device (VtBlob).
template <typename T, int N, int N_OPS>
void compact(const std::vector<T>& full, T* out) {
    constexpr int OPS = VtBlob<T>::ops(N_OPS), PER = VtBlob<T>::PER;
    std::copy(full.begin(), full.begin() + OPS, out);
    for (int i = N_OPS; i < N; ++i)
        for (int g = 0; g < 4; ++g)
            out[OPS + g * VtBlob<T>::row(N, N_OPS) + (i - N_OPS)] =
                full[((size_t)(i / PER) * 64 + 16 * g) * PER + i % PER];
}

template <typename T>
void build_all(const float* theta, int kbar, std::vector<T>& out) {
    using B = VtBlobs<T>;
    using L = VtLayout<T>;
    out.assign(B::size(kbar), (T)0);
    for (int k = 0; k < kbar; ++k) {
        const Wts w{theta + (size_t)k * BLOCK_W};
        std::vector<T> main(L::N_MAIN * 64, (T)0), sender(L::N_Q * 64, (T)0);
        build_main<T>(w, main.data());
        build_sender<T>(w, sender.data());
        compact<T, L::N_MAIN, L::N_OPS>(main, out.data() + (size_t)k * B::MAIN);
        compact<T, L::N_Q, L::N_QOPS>(sender, out.data() + (size_t)kbar * B::MAIN + (size_t)k * B::Q);
    }
    build_dec<T>(Wts{theta + (size_t)(kbar - 1) * BLOCK_W}, out.data() + (size_t)kbar * (B::MAIN + B::Q));
}

}  // namespace

void build_vt_maps(const float* one_block, std::vector<float>& main, std::vector<float>& sender,
                   std::vector<float>& dec) {
    using L = VtLayout<float>;
    const Wts w{one_block};
    main.assign(L::N_MAIN * 64, 0.0f);
    sender.assign(L::N_Q * 64, 0.0f);
    dec.assign(L::N_DEC * 64, 0.0f);
    build_main<float>(w, main.data());
    build_sender<float>(w, sender.data());
    build_dec<float>(w, dec.data());
}

void build_vt_blobs(const float* theta, int kbar, std::vector<double>& b64, std::vector<float>& b32) {
    build_all<double>(theta, kbar, b64);
    build_all<float>(theta, kbar, b32);
}

namespace {
unsigned lanes_grid(int n_tiles) { return (unsigned)(((int64_t)n_tiles * VT_TILE + VT_BLOCK - 1) / VT_BLOCK); }
}  // namespace

hipError_t launch_vt_nodes(const DevProb* tab, const VtTile* info, int n_tiles, int2* node, int32_t* pos,
                           hipStream_t s) {
    if (n_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(vt_nodes_kernel, dim3(lanes_grid(n_tiles)), dim3(VT_BLOCK), 0, s, tab, info, n_tiles, node, pos);
    return hipGetLastError();
}

hipError_t launch_vt_edges(const DevProb* tab, const VtTile* info, int n_tiles, const int2* node, const int32_t* pos,
                           VtRec<float>* rec32, VtRec<double>* rec64, hipStream_t s) {
    if (n_tiles <= 0) return hipSuccess;
    const dim3 grid(lanes_grid(n_tiles)), block(VT_BLOCK);
    if (rec32) hipLaunchKernelGGL(vt_edges_kernel<float>, grid, block, 0, s, tab, info, n_tiles, node, pos, rec32);
    if (rec64) hipLaunchKernelGGL(vt_edges_kernel<double>, grid, block, 0, s, tab, info, n_tiles, node, pos, rec64);
    return hipGetLastError();
}

hipError_t launch_vt_fill(double* p, int64_t n, double v, hipStream_t s) { return fill<double>(p, n, v, s); }
hipError_t launch_vt_fill(float* p, int64_t n, float v, hipStream_t s) { return fill<float>(p, n, v, s); }

namespace {
template <typename T>
void blocks(const DevProb* tab, const int4* tiles, int n_tiles, bool solo, int kbar, double alpha, int apply,
            const T* blobs, hipStream_t s) {
    using B = VtBlobs<T>;
    const T* q = blobs + (size_t)kbar * B::MAIN;
    const T* dec = blobs + (size_t)kbar * (B::MAIN + B::Q);
    constexpr int W = BLOCK / 64, WG_MAX = N_CU * WG_PER_CU;
    int grid = (n_tiles + W - 1) / W;
    grid = grid > WG_MAX ? WG_MAX : grid;
    grid = (grid + N_XCD - 1) / N_XCD * N_XCD;
    for (int k = 0; k < kbar; ++k) {
        VtArgs<T> a{tab, tiles, n_tiles, solo ? 1 : 0, apply, k & 1, (T)alpha, blobs + (size_t)k * B::MAIN, nullptr};
        if (k + 1 < kbar) {
            a.next = q + (size_t)(k + 1) * B::Q;
            hipLaunchKernelGGL((dss_block_kernel<T, false>), dim3(grid), dim3(BLOCK), 0, s, a);
        } else {
            a.next = dec;
            hipLaunchKernelGGL((dss_block_kernel<T, true>), dim3(grid), dim3(BLOCK), 0, s, a);
        }
    }
}
}  // namespace

template <typename T>
hipError_t launch_dss_tiles(const DevProb* tab, const int2* subs, int n_subs, const int4* tiles, int n_tiles,
                            bool solo, int kbar, double alpha, int apply, const T* blobs, hipStream_t s, bool check) {
    if (n_subs <= 0 || n_tiles <= 0) return hipSuccess;
    using B = VtBlobs<T>;
    const T* q = blobs + (size_t)kbar * B::MAIN;
    hipLaunchKernelGGL(dss_restrict_kernel<T>, dim3(n_subs), dim3(RB), 0, s, tab, subs, q, apply);
    blocks<T>(tab, tiles, n_tiles, solo, kbar, alpha, apply, blobs, s);
    return check ? hipGetLastError() : hipSuccess;
}
template hipError_t launch_dss_tiles<double>(const DevProb*, const int2*, int, const int4*, int, bool, int, double,
                                             int, const double*, hipStream_t, bool);
template hipError_t launch_dss_tiles<float>(const DevProb*, const int2*, int, const int4*, int, bool, int, double, int,
                                            const float*, hipStream_t, bool);

}  // namespace ddmgnn
