// Device-side types shared by the kernel translation units and the host
// runtime: Krylov scalars, the per-problem pointer table, work items and the
// kernel launchers.
//
// Every kernel is table driven. A launch serves one or several problems (a
// batch): workgroup b looks up its work item (problem index, sub-mesh / row /
// local workgroup) and reads that problem's pointers from the table. A single
// solve is a batch of one. Problems that have converged keep their slots in
// the grid but their workgroups return at once (the per-problem done flag).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

namespace ddmgnn {

constexpr int D = 10;           // latent width of the paper's model (Sec. IV.B); the MFMA kernel's width
constexpr int MAX_M = 4;        // largest FCG truncation supported
constexpr int MAX_RESTART = 64; // largest FGMRES cycle
constexpr int VEC_BLOCK = 256;  // threads of the vector kernels
constexpr int VEC_GRID = 1024;  // max workgroups per problem in the vector kernels
constexpr int N_XCD = 8;        // accelerator dies; workgroups are dispatched to them round-robin
constexpr int DSS_BLOCK = 512;  // threads of the VALU DSS kernel
constexpr int DSS_WIDE_BLOCK = 1024;  // its form for launches of fewer sub-meshes than compute units
constexpr int N_CU = 256;  // compute units of an MI355X
constexpr size_t LDS_LIMIT = 160 * 1024;

// Rows of a problem's partial sums: the prolongation's dots, <p, A p> and <p, r>, |r|^2.
// A kernel that completes another's sums writes its own to other rows.
constexpr int PART_PROLONG = 0, PART_SPMV = MAX_M + 1, PART_UPDATE = MAX_M + 3, N_PART = MAX_M + 4;

// Krylov scalars of one problem, resident in device memory.
struct KState {
    double r0n;            // |r_0|
    double rtol;
    double rel;            // |r_it| / |r_0|
    double beta;           // CG: p_new = r + beta p
    double pq[MAX_M + 1];  // <p, A p> of each direction-ring slot
    double rho;            // PCG/CG: <r, z> of the current iteration
    double rr_true;        // |b - A u|^2 at exit
    int it;                // completed iterations
    int done;
    int status;
    int max_it;            // the update kernel raises done once it reaches max_it
    // FGMRES cycle (unused by the other methods)
    double gm_beta;        // |r| at the start of the cycle
    double gm_hnext;       // h_{j,j-1}: norm of the unnormalised basis vector j
    int gm_j;              // step of the cycle (basis vectors 0..gm_j exist)
    int gm_k;              // steps of a finished cycle
    int gm_end;            // the cycle is over: update u, restart or stop
    int gm_conv;           // the residual estimate met the tolerance
};

// Per slot position in tile order (nodes of a sub-mesh by decreasing
// in-degree): the node's local id, in-degree, first padded in-edge record, and the bf16 bits
// of its sub-mesh-centred coordinates split as x = x_hi + x_lo, y = y_hi + y_lo.
struct TileNode {
    int32_t e0;
    uint16_t j;
    uint16_t deg;
    uint16_t xh, xl, yh, yl;
};
static_assert(sizeof(TileNode) == 16, "tile record layout");

// Arrays of the tiled DSS forward in one precision (dss_tile.hip): an in-edge
// (sender's tile lane, distance) per edge row and node of a tile, the per-tile
// latent states, and the two sender-row buffers.
template <typename T>
struct VtRec;
template <>
struct VtRec<float> {
    int32_t src;
    float nd;
};
template <>
struct VtRec<double> {
    int32_t src, pad;
    double nd;
};
template <typename T>
struct VtVecs {
    const VtRec<T>* rec;
    T* info;  // FP32: per tile and node (x, y, in-degree, c); FP64: unused
    T* h;     // per tile and lane: three components, and (FP64) c or the in-degree
    T* q[2];  // 20 values per tile lane; the last row is the sentinel (-inf)
};

// Device view of one problem (all pointers device memory).
struct DevProb {
    // matrix, right-hand side, boundary
    const int32_t* rowptr;
    const int32_t* col;
    const double* val;
    const double* b;
    const double* u0;
    const uint8_t* dirichlet;
    // decomposition and DSS graphs (slot = position in sub_nodes)
    const int32_t* sub_ptr;
    const int32_t* sub_nodes;
    const double* weights;
    const int32_t* edge_ptr;    // per slot, in-edge range (global edge index)
    const uint16_t* edge_src;   // per edge, sender local id; padded by 8 entries
    const float* edge_nd;       // per edge, |d_jl|; padded by 8 entries
    const uint32_t* erec;       // per node of each sub-mesh, its in-edges (FP16 |d_jl| | 20 * sender << 16)
                                // padded with sentinel records (sender k_i, |d| 0) to a multiple of MFMA_EC
    const int32_t* epad_sub;    // [K + 1] range of each sub-mesh in erec
    const TileNode* tiles;      // per slot position in tile order (e0 indexes erec)
    const double* xy64;         // per slot, raw coordinates
    const float* xyc32;         // per slot, sub-mesh-centred coordinates
    // tiles of 16 nodes of the FP64 and FP32 DSS forward (width 10; null until its first use)
    const int32_t* vt_first;    // [K] first tile of each sub-mesh
    const int2* vt_node;        // per tile and lane: slot (-1: none), in-degree
    VtVecs<double> vt64;
    VtVecs<float> vt32;
    const int32_t* node_ptr;    // per node, range of its slots
    const int32_t* node_slots;
    const int32_t* slot_sub;
    const double* a0inv;        // K x K
    double* lu_inv;             // local exact solves: per sub-mesh (R_i A R_i^T)^{-1} (lu_dense), or the
                                // tiles of its negative and their units' partial products
    const int64_t* lu_off;      // [2 K] offsets of both in lu_inv (null until built)
    // iteration vectors
    double* u;
    double* r;                  // residual; input of the apply
    double* z;                  // output of the apply
    const double* c_in;         // DSS forward entry: per-slot inputs (null in solves)
    double* p[MAX_M + 1];       // direction ring
    double* q[MAX_M + 1];       // A p of each ring slot
    double* s;                  // [K] |R_i r|
    double* y0;                 // [K] R_0 r
    double* y;                  // [K] coarse solution
    double* local;              // per slot, |R_i r| r~_i (or r~_i for the forward entry)
    double* qg64;               // DSS fallback storage when LDS is too small (may be null)
    double* hg64;               // FP64 DSS latent state
    float* qg32;
    float* hg32;                // FP32 latent state of sub-meshes beyond the register-resident size
    double* c64;                // normalised local right-hand sides of those sub-meshes (FP64 form),
    float* c32;                 // and the same storage read as FP32 (FP32 form)
    KState* st;                 // null: no Krylov scalars, no done flag
    double* partials;           // N_PART x VEC_GRID per-workgroup partial sums
    // FGMRES storage (null until a problem is solved with FGMRES)
    double* gm_v;               // (restart + 1) x n: Arnoldi basis V
    double* gm_z;               // restart x n: preconditioned vectors Z = M(V)
    double* gm_part;            // (restart + 1) x VEC_GRID partial sums of the Gram passes
    double* gm_small;           // H [(restart + 1) x restart, column j at j * (restart + 1)],
                                // cs, sn [restart], g [restart + 1], y [restart], tmp [restart + 1]
    double rtol;                // read by the init kernel
    int max_it;
    int n;
    int K;
    int nblk;                   // workgroups of this problem in the vector kernels
};

// Options of one Krylov iteration, common to the problems of a launch.
struct IterArgs {
    int mode;        // DDMGNN_FCG / PCG / CG / FGMRES; < 0: bare apply (no Krylov scalars)
    int m;           // directions kept (FCG m_max; 1 for PCG and CG); FGMRES: cycle length
    int unweighted;  // gluing without partition-of-unity weights
    int coarse;      // add the coarse correction
};

// Ring slots of iteration `it` with `m` kept directions: the new direction
// goes to it % (m+1), previous direction k (0 = most recent) is in (it-1-k) mod (m+1).
__host__ __device__ inline int ring_cur(int it, int m) { return it % (m + 1); }
__host__ __device__ inline int ring_prev(int it, int m, int k) {
    const int nr = m + 1;
    return ((it - 1 - k) % nr + nr) % nr;
}

// Launchers (kernels.hip). tab: device table; the int2 lists are device
// arrays of (problem, item) pairs, one per workgroup. check = false skips
// hipGetLastError (not allowed while a stream is being captured).
hipError_t prepare_dss_valu(int precision, int d, size_t shmem);
hipError_t launch_dss_valu(const DevProb* tab, const int2* work, int n_work, int precision, int d, bool qlds,
                           int kbar, double alpha, int apply, const float* theta32, const double* theta64,
                           size_t shmem, hipStream_t s, bool check);
// The VALU DSS forward for sub-meshes of more than kMaxSubNodes nodes (h, c
// and Q in the per-slot global buffers hg32/hg64, c32/c64, qg32/qg64).
hipError_t launch_dss_big(const DevProb* tab, const int2* work, int n_work, int precision, int d, int kbar,
                          double alpha, int apply, const float* theta32, const double* theta64, hipStream_t s,
                          bool check);
// Exact local solves (DDM-LU): restriction as in the DSS kernels, then
// local = (R_i A R_i^T)^{-1} R_i r per sub-mesh. A small one (lu_dense) is one workgroup's
// (unit -1) and held as a square of row stride lu_ld(k). A larger one, of nt
// rows of tiles, is shared by lu_units workgroups (unit u: rows u and nt - 1 - u, nt + 1
// tiles), whose partial products a second kernel adds. units: (problem, sub-mesh, unit);
// those of sub-meshes of at most LU_LDS_K nodes, and the larger ones (big); max_k: largest
// sub-mesh of each list (dynamic LDS). subs: (problem, sub-mesh) of those in tiles.
// prepare_lu_local raises the kernels' LDS limits (not allowed during capture).
constexpr int LU_LDS_K = 2048, LU_DENSE_K = 256, LU_DENSE_MIXED = 202;
// Whether the inverse of a sub-mesh of k nodes is held as a square; max_k: the problem's
// largest. Up to LU_DENSE_MIXED nodes tiles may hold more bytes than the square (k <= 63,
// 65-110, 129-156, 193-202: at 16 nodes 16 times, at 65 three times), and never beyond.
// Where every sub-mesh of a problem is a square the second kernel is not needed either,
// which pays to LU_DENSE_K. Per launch, squares against tiles: 40 sub-meshes of up to 64
// nodes 5.3 and 7.5 us, of up to 248 8.3 and 9.8, of up to 326 11.6 and 10.9; 1200 of up to
// 58 8.2 and 16.9, up to 202 26.4 and 30.0, of 40 to 540 (both forms) 143 and 141.
inline bool lu_dense(int k, int max_k) { return k <= (max_k <= LU_DENSE_K ? LU_DENSE_K : LU_DENSE_MIXED); }
__host__ __device__ inline int lu_units(int k) { return ((k + 63) / 64 + 1) / 2; }
struct LuWork {
    const int4* units;
    int n_units, max_k;
    const int4* big;
    int n_big, max_k_big;
    const int2* subs;
    int n_subs;
};
hipError_t prepare_lu_local();
hipError_t launch_lu_local(const DevProb* tab, const LuWork& w, hipStream_t s, bool check);
// Device factorisation (factor.hip) of symmetric matrices held as the SYM_TILE x
// SYM_TILE tiles of their lower triangle. launch_lu_assemble: the tiles (zeroed
// before) of A_i = R_i A R_i^T, those of sub-mesh subs[m] at base + off[m].
// launch_lu_small: (R_i A R_i^T)^{-1} of sub-meshes of at most SYM_TILE nodes as squares
// at out + lu_off[i]; launch_lu_pack: squares from the inverted tiles of larger ones.
// launch_coarse_assemble:
// A_0 = R_0 A R_0^T (K x K, deterministic summation order), symmetrised, its diagonal
// copied to diag0. launch_gj_invert: in-place -A^{-1} of a batch of SPD matrices (matrix
// m's tiles at base + off[m], orders and prefixes of plan.meta in meta) over the
// whole device; scratch holds plan.scratch_doubles(). launch_coarse_invert: A_0^{-1} in
// place of A_0 (K x K); scratch holds coarse_scratch_doubles(K). *status (device,
// zeroed by the caller) gets bit 0 when a pivot is not positive (coarse: not above
// 1e-12 of its original diagonal entry).
constexpr int SYM_TILE = 64;
__host__ __device__ inline int64_t sym_tile(int I, int J) {  // offset of tile (I, J), J <= I
    return ((int64_t)I * (I + 1) / 2 + J) * SYM_TILE * SYM_TILE;
}
__host__ __device__ inline int64_t sym_doubles(int64_t k) {
    const int64_t nt = (k + SYM_TILE - 1) / SYM_TILE;
    return nt * (nt + 1) / 2 * SYM_TILE * SYM_TILE;
}
struct GjPlan {
    int nm = 0, steps = 0;
    int64_t n_rows = 0, n_tiles = 0;  // tiles per column of all matrices, and all tiles
    std::vector<int32_t> meta;        // orders, prefix of the tiles per column, prefix of the tiles
    explicit GjPlan(const std::vector<int32_t>& k);
    size_t scratch_doubles() const;
};
struct LuMatrix {  // a problem's matrix and sub-meshes
    const int32_t* rowptr;
    const int32_t* col;
    const double* val;
    const int32_t* sub_ptr;
    const int32_t* sub_nodes;
};
hipError_t launch_lu_assemble(const LuMatrix& a, const int32_t* subs, int n, const int64_t* off, double* base,
                              hipStream_t s);
hipError_t launch_lu_small(const LuMatrix& a, const int32_t* subs, int n, const int64_t* lu_off, double* out,
                           int* status, hipStream_t s);
hipError_t launch_lu_pack(const int32_t* sub_ptr, const int32_t* subs, int n, const int64_t* off, const double* base,
                          const int64_t* lu_off, double* out, hipStream_t s);
hipError_t launch_coarse_assemble(const int32_t* rowptr, const int32_t* col, const double* val,
                                  const int32_t* sub_ptr, const int32_t* sub_nodes, const double* weights,
                                  const int32_t* node_ptr, const int32_t* node_slots, const int32_t* slot_sub, int K,
                                  double* a0, double* diag0, hipStream_t s);
hipError_t launch_gj_invert(const GjPlan& plan, const int32_t* meta, double* base, const int64_t* off, double* scratch,
                            int* status, hipStream_t s);
size_t coarse_scratch_doubles(int K);
hipError_t launch_coarse_invert(double* a0, int K, const double* diag0, double* scratch, int* status, hipStream_t s);
// Overlap expansion on the device (overlap.hip). OV_CAP: most sub-meshes a node
// may belong to; OV_SORT_MAX: largest sub-mesh the per-part sort holds (the
// library's sub-mesh limit). ov_check: bit 0 of *status for a triangle node id
// out of [0, n), bit 1 for a part id out of [0, n_part). ov_grow: node ->
// triangle lists (tri_cnt must be zero), then delta rounds of growth of the
// per-node part sets (bit 2 of *status on overflow); *sets_out / *sz_out point
// at the final sets. ov_count: sub-mesh sizes (part_cnt zero) and their
// exclusive scan sub_ptr[0..n_part]. ov_fill: the sorted lists and weights
// (part_cur zero).
constexpr int OV_CAP = 16;
constexpr int OV_SORT_MAX = 16384;
hipError_t ov_check(const int32_t* tri, int64_t n_tri, const int32_t* part, int64_t n, int32_t n_part, int* status,
                    hipStream_t s);
hipError_t ov_grow(const int32_t* tri, int64_t n_tri, const int32_t* part, int64_t n, int32_t delta,
                   int32_t* tri_cnt, int64_t* tri_ptr, int32_t* tri_list, int32_t* sets0, int32_t* sets1,
                   uint8_t* sz0, uint8_t* sz1, int32_t** sets_out, uint8_t** sz_out, int* status, hipStream_t s);
hipError_t ov_count(const int32_t* sets, const uint8_t* sz, int64_t n, int32_t n_part, int32_t* part_cnt,
                    int64_t* sub_ptr, hipStream_t s);
hipError_t ov_fill(const int32_t* sets, const uint8_t* sz, int64_t n, const uint8_t* dirichlet, int32_t n_part,
                   const int64_t* sub_ptr, int64_t sk, int32_t* part_cur, int32_t* nodes, double* weights,
                   hipStream_t s);
// Writes a one-problem table.
hipError_t launch_set_view(DevProb* at, const DevProb& v, hipStream_t s);
hipError_t launch_coarse(const DevProb* tab, const int2* rows, int n_rows, hipStream_t s, bool check);
hipError_t launch_prolong(const DevProb* tab, const int2* blk, int n_blk, const IterArgs& it, hipStream_t s,
                          bool check);
// The launchers below end with a finalize launch of one workgroup per
// problem: n_prob = all problems of the table, or the problems of `list`.
// FGMRES: one step of every problem of the table (after its apply) and the
// normalisation that starts the next step (before it).
hipError_t launch_fgmres_next(const DevProb* tab, const int2* blk, int n_blk, const IterArgs& it, hipStream_t s,
                              bool check);
hipError_t launch_fgmres_step(const DevProb* tab, const int2* blk, int n_blk, int n_prob, const IterArgs& it,
                              hipStream_t s, bool check);
hipError_t launch_krylov(const DevProb* tab, const int2* blk, int n_blk, int n_prob, const IterArgs& it,
                         hipStream_t s, bool check);
hipError_t launch_init(const DevProb* tab, const int2* blk, int n_blk, const int* list, int n_list, hipStream_t s);
hipError_t launch_resid(const DevProb* tab, const int2* blk, int n_blk, const int* list, int n_list, hipStream_t s);
hipError_t launch_gather_states(const DevProb* tab, int n, KState* out, hipStream_t s);
// Entry points: y = A x with the solve's grouped SpMV over nblk workgroups, and
// *out = x.y (device) with the solve's two-kernel reduction (partials: VEC_GRID
// doubles of scratch); n < 2^31.
hipError_t launch_spmv(const int32_t* rowptr, const int32_t* col, const double* val, const double* x, double* y,
                       int n, int nblk, hipStream_t s);
hipError_t launch_dot(const double* x, const double* y, int n, double* partials, double* out, hipStream_t s,
                      bool check);

// Allocation-free entry points (noalloc.hip): a static device array of
// NOALLOC_SCRATCH_DOUBLES doubles per device holds their scratch. noalloc_init
// looks up the array's device address on the current device (once per device);
// noalloc_scratch returns it (nullptr before noalloc_init ran on that device).
constexpr int NOALLOC_SCRATCH_DOUBLES = VEC_GRID;  // the dot product's partial sums
hipError_t noalloc_init(int device);
double* noalloc_scratch(int device);

// Training of DSS_theta (train.hip), in tiles of 16 nodes of all samples (d = D).
constexpr int TRAIN_BLOCK = 1024;                       // threads of the reductions
constexpr int TRAIN_NWB = 11 * D * D + 15 * D + 1;      // weights per block
constexpr int TRAIN_BLOB = (56 + 16 + 12 + 32 + 28) * 64;  // values of a block's blob
constexpr int TRAIN_ACC = 56;                           // accumulators per lane of the backward pass
// An edge of a tile's node: the other end's tile lane of the problem (-1: none),
// d = x_send - x_recv and |d|.
struct TrainEdge {
    int32_t node;
    float dx, dy, nd;
};
// Where a weight's gradient lies in the accumulators of a backward launch: that of its
// block, or the next one (edges); the sum of `lanes` consecutive values.
struct TrainEntry {
    int32_t at;
    int16_t lanes;
    int8_t edges, negative;
};
struct TrainEdgeArgs {
    const int4* info;          // tiles of the problem (dss_tile.h)
    const int2* out_rows;      // per tile: first out-edge row, rows
    int n_tiles;
    const int2* node;          // per tile lane: slot (-1: none), in-degree
    const int32_t* pos;        // per slot, its tile lane
    const int32_t* edge_ptr;
    const uint16_t* edge_src;
    const float* edge_nd;
    const int32_t* oe_ptr;     // per slot, range of its out-edges
    const int32_t* oe_edge;    // the in-edge index of each out-edge
    const uint16_t* oe_recv;   // its receiver's local id
    const double* xy64;        // per slot, coordinates
    TrainEdge* rin;
    TrainEdge* rout;
};
struct TrainArgs {
    // tiles of the samples: (tile of the problem, batch lane - problem lane, first in-edge
    // row, rows), (first out-edge row, rows, offset of the right-hand side in c)
    const int4* items;
    int n_tiles;
    int kbar;
    int ks;                    // values per tile lane in r, rho and gr (>= kbar)
    float alpha;
    const int4* info;
    const int2* node;
    const int32_t* pos;
    const TrainEdge* rin;
    const TrainEdge* rout;
    const int32_t* lm_ptr;     // per slot, range of its row of A_i = R_i A R_i^T
    const uint16_t* lm_col;    // local column
    const float* lm_val;
    const float* c;
    const float* blobs;        // per block, TRAIN_BLOB values
    float* blobs_out;          // the same, written first
    float2* in;                // per tile lane: c, in-degree
    float* h;                  // [kbar + 1] latent states of every tile
    float* q;                  // [kbar] sender rows (20 per tile lane and a sentinel)
    float* m;                  // [kbar] message hidden sums
    float* r;                  // decoded states, residuals, dL/dr: per tile lane, ks blocks
    float* rho;
    float* gr;
    float* pg[2];              // receiver rows: receiver part and message gradient
    float* own;                // the same in lane order, with dL/dH
    float* part;               // per backward launch and workgroup, its accumulators
    double* sse;               // per workgroup of the residual kernel
};
// Most tiles of the samples run together: they share one scratch region, of 4 GB at 30 blocks.
// A third of them (1.3 GB) costs 16% at 400 samples of 900 nodes (6.4 and 7.5 ms) and 5% at
// 2500; they are halved only where the region cannot be allocated.
constexpr int64_t TRAIN_TILES = 32768;
void build_train_maps(std::vector<int32_t>& map, std::vector<TrainEntry>& ent);
int64_t train_sse_count(int64_t tiles, int ks);
int train_workgroups(int64_t tiles);
hipError_t launch_train_edges(const TrainEdgeArgs& a, hipStream_t s);
// Forward, backward and the accumulators' sums in red ([kbar + 1][TRAIN_ACC * 64], added to when `add`).
hipError_t launch_train_grad(const TrainArgs& a, const float* theta, const int32_t* map, double* red, bool add,
                             hipStream_t s);
// grad = scale * the sums; out2[0] = |grad|^2, out2[1] = sum of sse.
hipError_t launch_train_reduce(const double* red, const TrainEntry* ent, int kbar, double scale, float* grad,
                               double* out2, const double* sse, int n_sse, hipStream_t s);
hipError_t launch_adam(float* theta, const float* grad, float* m, float* v, int64_t n, float gscale, float lr,
                       float b1, float b2, float bc1, float bc2, float eps, hipStream_t s);
// r = b - A u, then c = R_i r / |R_i r| per sub-mesh (slot order).
hipError_t launch_train_rhs(const int32_t* rowptr, const int32_t* col, const double* val, const double* bb,
                            const double* u, double* r, int n, const int32_t* sub_ptr, const int32_t* sub_nodes,
                            int K, float* c, hipStream_t s);

// Workgroups a problem of n rows takes in the vector kernels.
// Workgroups of a problem in the vector kernels: one per VEC_BLOCK rows up to
// VEC_GRID, rounded up to a multiple of N_XCD (so that a problem's workgroups
// start on die 0 in every launch and split evenly over the dies).
inline int vec_blocks(int64_t n) {
    int64_t g = (n + VEC_BLOCK - 1) / VEC_BLOCK;
    g = g > VEC_GRID ? VEC_GRID : g;
    g = (g + N_XCD - 1) / N_XCD * N_XCD;
    return (int)(g < N_XCD ? N_XCD : g);
}
static_assert(VEC_GRID % N_XCD == 0, "vector grid must split over the dies");

}  // namespace ddmgnn
