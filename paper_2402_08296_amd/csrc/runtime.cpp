// Host runtime of the DDM-GNN solver: contexts, models, problems, batches of
// problems solved in lockstep, the solve driver (graph-captured chunks of
// iterations, host polls of the per-problem converged flags) and the C ABI
// declared in include/ddmgnn.h (the serving entry points are in server.cpp).
#include "runtime.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>

namespace ddmgnn {

namespace {
thread_local std::string g_err;
std::atomic<uint64_t> g_next_id{1};
}  // namespace

int fail(int code, const std::string& msg) {
    g_err = msg;
    return code;
}

// ------------------------------------------------------------------ batch
// Sub-meshes of a batch that the FP64 / FP32 forward runs (those of at most kMaxSubNodes).
struct DssSide {
    std::vector<int2> host;            // (problem, sub-mesh) by decreasing size
    DevBuf<int2> work;                 // the same
    int n = 0, max_k = 0;
    int64_t tiles = 0;                 // tiles of 16 nodes
    // Built at the first use in tiles (d = 10): the tiles by problem and sub-mesh, and, where a
    // problem is untiled, the sub-meshes of the others (subs) and of the untiled ones (plain).
    std::vector<uint8_t> untiled;      // of each problem, as these lists were built
    DevBuf<int4> items;
    DevBuf<int2> subs, plain;
    int n_items = 0, n_subs = 0, n_plain = 0, max_k_plain = 0;
};

struct Batch {
    ddmgnn_ctx* ctx = nullptr;
    std::vector<ddmgnn_problem*> probs;
    std::vector<uint64_t> ids;
    std::shared_ptr<ModelDev> model;
    std::vector<DevProb> views;        // host copy of tab
    DevBuf<DevProb> tab;               // table of the solve
    DevBuf<DevProb> hook;              // one-problem table of the entry points that redirect vectors
    // DSS work lists, (problem, sub-mesh) by decreasing sub-mesh size:
    // those that fit the MFMA kernel; the others; of all, those of at most kMaxSubNodes.
    // (work_big: sub-meshes beyond kMaxSubNodes, which run the global-memory form of the VALU
    // kernel in every precision)
    DssSide valu, rest;                // all, and those that the MFMA kernel does not run
    DevBuf<int2> work_mfma, work_big;
    std::vector<int2> all;             // host: every sub-mesh
    int n_mfma = 0, n_big = 0;
    // the MFMA list split by workgroup size: sub-meshes that run two per compute
    // unit in MFMA_SMALL_BLOCK-thread workgroups, and the rest; dynamic LDS of each launch
    DevBuf<int2> work_mfma_small;
    int n_mfma_small = 0;
    size_t lds_mfma = 0, lds_mfma_small = 0;
    int max_k_all = 0;
    // exact local solves (built at the first one): units of valu's and work_big's
    // sub-meshes, and the sub-meshes whose inverses are held in tiles
    bool lu_ready = false;
    DevBuf<int4> lu_small, lu_big;
    DevBuf<int2> lu_subs;
    int n_lu_small = 0, n_lu_big = 0, n_lu_subs = 0;
    DevBuf<int2> vec_blk;              // (problem, local workgroup)
    int n_vec = 0;
    DevBuf<int2> coarse_rows;          // (problem, row)
    int n_coarse = 0;
    DevBuf<int2> sub_blk;              // subset of vec_blk (init and residual of some problems)
    int n_sub_blk = 0;
    DevBuf<int> sub_list;              // the problems of that subset (their finalize workgroups)
    int n_sub_list = 0;
    DevBuf<KState> st_gather;
    KState* host_st = nullptr;         // pinned, one per problem
    // captured chunks of iterations: of check_every of them, and a short one (brief_chunk)
    struct Graph {
        hipGraphExec_t exec = nullptr;
        uint64_t key = 0;
        void reset() {
            if (exec) (void)hipGraphExecDestroy(exec);
            exec = nullptr;
            key = 0;
        }
    } graph, brief;
    int last_it = 0;                   // iterations of the last solve
    ~Batch() {
        graph.reset();
        brief.reset();
        if (host_st) (void)hipHostFree(host_st);
    }
};

namespace {

DevProb make_view(ddmgnn_problem* P) {
    DevProb v{};
    v.rowptr = P->rowptr.p; v.col = P->col.p; v.val = P->val.p; v.b = P->b.p; v.u0 = P->u0.p;
    v.dirichlet = P->dirichlet.p;
    v.sub_ptr = P->sub_ptr.p; v.sub_nodes = P->sub_nodes.p; v.weights = P->weights.p;
    v.edge_ptr = P->edge_ptr.p; v.edge_src = P->edge_src.p; v.edge_nd = P->edge_nd.p; v.erec = P->erec.p;
    v.epad_sub = P->epad_sub.p;
    v.tiles = P->tiles.p; v.xy64 = P->xy64.p; v.xyc32 = P->xyc32.p;
    v.vt_first = P->vt_first_dev; v.vt_node = P->vt_node; v.vt64 = P->vt64.v; v.vt32 = P->vt32.v;
    v.node_ptr = P->node_ptr.p; v.node_slots = P->node_slots.p; v.slot_sub = P->slot_sub.p; v.a0inv = P->a0inv.p;
    v.lu_inv = P->lu_inv.p; v.lu_off = P->lu_off.p;
    v.gm_v = P->gm_v.p; v.gm_z = P->gm_z.p; v.gm_part = P->gm_part.p; v.gm_small = P->gm_small.p;
    v.u = P->u.p; v.r = P->r.p; v.z = P->z.p; v.c_in = nullptr;
    const int64_t n = P->hs.n;
    for (int i = 0; i <= MAX_M; ++i) {
        v.p[i] = P->ring.p + (size_t)i * n;
        v.q[i] = P->ring.p + (size_t)(MAX_M + 1 + i) * n;
    }
    v.s = P->s.p; v.y0 = P->y0.p; v.y = P->y.p; v.local = P->local.p;
    v.qg64 = P->qglobal64.p; v.hg64 = P->hglobal64.p; v.qg32 = P->qglobal32.p;
    v.hg32 = P->hglobal32.p; v.c64 = P->cglobal.p; v.c32 = reinterpret_cast<float*>(P->cglobal.p);
    v.st = P->st.p;
    v.partials = P->partials.p;
    v.rtol = P->rtol;
    v.max_it = P->max_it;
    v.n = (int)n;
    v.K = P->hs.K;
    v.nblk = problem_vec_blocks(P);
    return v;
}

hipError_t upload_async(void* dst, const void* src, size_t bytes, hipStream_t s) {
    if (bytes == 0) return hipSuccess;
    hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    return hipStreamSynchronize(s);
}

template <typename T>
int upload_list(DevBuf<T>& buf, const std::vector<T>& v, hipStream_t s) {
    if (buf.n < v.size() || !buf.p) HIP_TRY(buf.alloc(std::max<size_t>(v.size(), 1)));
    HIP_TRY(upload_async(buf.p, v.data(), v.size() * sizeof(T), s));
    return DDMGNN_OK;
}

bool valu_q_in_lds(int max_k, int precision, int d) {
    const size_t esz = precision == DDMGNN_FP64 ? sizeof(double) : sizeof(float);
    return (size_t)max_k * 2 * d * esz + 1024 <= LDS_LIMIT;
}

size_t valu_shmem(int max_k, int precision, int d) {
    const size_t esz = precision == DDMGNN_FP64 ? sizeof(double) : sizeof(float);
    return (size_t)max_k * 2 * d * esz;
}

// Whether an inversion's status word says that a pivot failed (waits for the stream).
int pivots_ok(const DevBuf<int>& status, hipStream_t s) {
    int bad = 0;
    HIP_TRY(hipMemcpyAsync(&bad, status.p, sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    return bad ? DDMGNN_E_NOT_SPD : DDMGNN_OK;
}

// Most doubles of tiles and panels while inverses that are kept as squares are formed.
constexpr int64_t LU_TEMP = 64 << 20;

// Exact local solves: the inverses of R_i A R_i^T, assembled from the problem's
// device matrix and inverted on the device.
int prepare_lu(ddmgnn_problem* P) {
    HIP_TRY(prepare_lu_local());
    if (P->lu_inv.p) return DDMGNN_OK;
    hipStream_t s = P->ctx->stream;
    const auto& hs = P->hs;
    const LuMatrix A{P->rowptr.p, P->col.p, P->val.p, P->sub_ptr.p, P->sub_nodes.p};
    std::vector<int64_t> off((size_t)hs.K * 2, 0);
    int64_t total = 0;
    // A group of sub-meshes inverted together: their tiles lie in lu_inv, or in a buffer from
    // which their squares are packed.
    struct Group {
        std::vector<int32_t> subs, k;
        std::vector<int64_t> at;  // offset of each one's tiles
        int64_t doubles = 0, temp = 0;
        size_t list = 0, meta = 0, off = 0;  // its arrays in the device lists
    };
    int max_k = 0;
    for (int32_t i = 0; i < hs.K; ++i) max_k = std::max(max_k, (int)(hs.sub_ptr[i + 1] - hs.sub_ptr[i]));
    std::vector<int32_t> lists;  // the sub-meshes of one tile, then of every group its sub-meshes and plan
    std::vector<Group> groups(1);  // the first: tiles in lu_inv
    // Tiles, then squares, then partial products: tiles start on a cache line, and partial
    // products between them cost a launch 2%.
    for (int32_t i = 0; i < hs.K; ++i) {
        const int32_t k = (int32_t)(hs.sub_ptr[i + 1] - hs.sub_ptr[i]);
        if (lu_dense(k, max_k)) continue;
        groups[0].subs.push_back(i);
        groups[0].k.push_back(k);
        groups[0].at.push_back(off[i] = total);
        total += sym_doubles(k);
    }
    groups[0].doubles = total;
    for (int32_t i = 0; i < hs.K; ++i) {
        const int32_t k = (int32_t)(hs.sub_ptr[i + 1] - hs.sub_ptr[i]);
        if (!lu_dense(k, max_k)) continue;
        off[i] = total;
        total += k * lu_ld(k);
        if (k <= SYM_TILE) {
            lists.push_back(i);
            continue;
        }
        const int64_t d = sym_doubles(k), t = d + (2 * ((k + SYM_TILE - 1) / SYM_TILE) + 1) * SYM_TILE * SYM_TILE;
        if (groups.size() == 1 || groups.back().temp + t > LU_TEMP) groups.emplace_back();
        Group& g = groups.back();
        g.subs.push_back(i);
        g.k.push_back(k);
        g.at.push_back(g.doubles);
        g.doubles += d;
        g.temp += t;
    }
    for (size_t q = 0; q < groups[0].subs.size(); ++q) {
        off[(size_t)hs.K + groups[0].subs[q]] = total;
        total += (int64_t)lu_units(groups[0].k[q]) * groups[0].k[q];
    }
    const int n_small = (int)lists.size();
    std::vector<GjPlan> plans;
    size_t n_tiles = 0, n_scratch = 0;
    for (Group& g : groups) {
        plans.emplace_back(g.k);
        const GjPlan& plan = plans.back();
        g.list = lists.size();
        lists.insert(lists.end(), g.subs.begin(), g.subs.end());
        g.meta = lists.size();
        lists.insert(lists.end(), plan.meta.begin(), plan.meta.end());
        g.off = off.size();
        off.insert(off.end(), g.at.begin(), g.at.end());
        if (!g.subs.empty()) n_scratch = std::max(n_scratch, plan.scratch_doubles());
        if (&g != &groups[0]) n_tiles = std::max(n_tiles, (size_t)g.doubles);
    }
    auto build = [&]() -> int {
        DevBuf<int32_t> d_lists;
        DevBuf<double> temp;  // panels, then the tiles of a packed group
        DevBuf<int> status;
        HIP_TRY(P->lu_off.upload(off.data(), off.size(), s));
        HIP_TRY(d_lists.upload(lists.data(), lists.size(), s));
        HIP_TRY(P->lu_inv.alloc((size_t)std::max<int64_t>(total, 1)));
        HIP_TRY(temp.alloc(n_scratch + n_tiles));
        HIP_TRY(status.alloc(1));
        HIP_TRY(hipMemsetAsync(status.p, 0, sizeof(int), s));
        for (size_t q = 0; q < groups.size(); ++q) {
            const Group& g = groups[q];
            const int n = (int)g.subs.size();
            if (n == 0) continue;
            double* const base = q ? temp.p + n_scratch : P->lu_inv.p;
            const int32_t* subs = d_lists.p + g.list;
            const int64_t* at = P->lu_off.p + g.off;
            HIP_TRY(hipMemsetAsync(base, 0, (size_t)g.doubles * sizeof(double), s));
            HIP_TRY(launch_lu_assemble(A, subs, n, at, base, s));
            HIP_TRY(launch_gj_invert(plans[q], d_lists.p + g.meta, base, at, temp.p, status.p, s));
            if (q) HIP_TRY(launch_lu_pack(P->sub_ptr.p, subs, n, at, base, P->lu_off.p, P->lu_inv.p, s));
        }
        HIP_TRY(launch_lu_small(A, d_lists.p, n_small, P->lu_off.p, P->lu_inv.p, status.p, s));
        const int rc = pivots_ok(status, s);
        if (rc == DDMGNN_E_NOT_SPD) return fail(rc, "a local matrix R_i A R_i^T is not positive definite");
        return rc;
    };
    if (int rc = build()) {  // leave no half-built inverses behind
        P->lu_inv.reset();
        P->lu_off.reset();
        return rc;
    }
    P->device_bytes += lu_bytes(hs);
    return DDMGNN_OK;
}

// The inverses of a batch's problems and the lists of its launches.
int prepare_exact(Batch& B, bool& changed) {
    for (ddmgnn_problem* P : B.probs) {
        changed = changed || !P->lu_inv.p;
        if (int rc = prepare_lu(P)) return rc;
    }
    if (B.lu_ready) return DDMGNN_OK;
    std::vector<int2> subs;
    std::vector<int4> small, big;
    std::vector<int> max_k(B.probs.size(), 0);
    auto size = [&](const int2& w) {
        const auto& sp = B.probs[w.x]->hs.sub_ptr;
        return (int)(sp[w.y + 1] - sp[w.y]);
    };
    for (const int2& w : B.all) max_k[w.x] = std::max(max_k[w.x], size(w));
    static_assert(LU_LDS_K == kMaxSubNodes, "valu holds the sub-meshes of the exact solves' LDS form");
    for (const int2& w : B.all) {
        const int k = size(w);
        if (lu_dense(k, max_k[w.x])) {
            small.push_back(make_int4(w.x, w.y, -1, 0));
            continue;
        }
        subs.push_back(w);
        for (int u = 0; u < lu_units(k); ++u) (k > LU_LDS_K ? big : small).push_back(make_int4(w.x, w.y, u, 0));
    }
    hipStream_t s = B.ctx->stream;
    if (int rc = upload_list(B.lu_subs, subs, s)) return rc;
    if (int rc = upload_list(B.lu_small, small, s)) return rc;
    if (int rc = upload_list(B.lu_big, big, s)) return rc;
    B.n_lu_subs = (int)subs.size();
    B.n_lu_small = (int)small.size();
    B.n_lu_big = (int)big.size();
    B.lu_ready = true;
    return DDMGNN_OK;
}

// Whether the BF16 MFMA kernel runs sub-mesh `sub` of P (the model has the
// paper's latent width and the sub-mesh fits the kernel's node and LDS budgets).
bool mfma_runs_sub(const ddmgnn_problem* P, int sub) {
    return P->model->mfma && P->mfma_need[(size_t)sub] <= MFMA_LDS_LIMIT;
}
// Whether every sub-mesh of P runs on the VALU kernels under BF16.
bool all_valu_bf16(const ddmgnn_problem* P) {
    for (int i = 0; i < P->hs.K; ++i)
        if (mfma_runs_sub(P, i)) return false;
    return true;
}
bool any_valu_bf16(const ddmgnn_problem* P) {
    for (int i = 0; i < P->hs.K; ++i)
        if (!mfma_runs_sub(P, i)) return true;
    return false;
}

int prepare_fgmres(Batch& B, int R, bool& changed) {
    for (ddmgnn_problem* P : B.probs) {
        if (P->gm_R >= R) continue;
        const size_t n = (size_t)P->hs.n;
        P->device_bytes -= P->gm_R ? fgmres_bytes(P->hs.n, P->gm_R) : 0;
        P->gm_R = 0;
        HIP_TRY(P->gm_v.alloc((size_t)(R + 1) * n));
        HIP_TRY(P->gm_z.alloc((size_t)R * n));
        HIP_TRY(P->gm_part.alloc((size_t)(R + 1) * VEC_GRID));
        HIP_TRY(P->gm_small.alloc((size_t)R * R + 6 * R + 2));
        P->gm_R = R;
        P->device_bytes += fgmres_bytes(P->hs.n, R);
        changed = true;
    }
    return DDMGNN_OK;
}

// Whether a launch of `tiles` tiles of 16 nodes of a width-d model runs the tiled forward
// (dss_tile.hip): every FP64 one, and the FP32 ones of up to VT_MAX_FP32 tiles. Larger FP32
// launches fill the chip with one workgroup per sub-mesh, whose sender rows stay in LDS, while
// the tiled form's outgrow the last-level cache and pass through HBM. Per forward, one workgroup
// per sub-mesh and tiled, sub-meshes of 900 nodes: 35k tiles 1,470 and 1,240 us, 54k 2,030 and
// 1,870, 60k 2,530 and 2,530, 64k 2,550 and 2,680, 89k 3,590 and 3,730; of 450: 62k 2,680 and
// 2,590, 73k 3,060 and 3,020; of 1,500: 59k 5,660 and 3,890. Both give the same bits. Other
// widths and sub-meshes beyond kMaxSubNodes run the kernels of kernels.hip.
bool runs_tiled(int d, int precision, int64_t tiles) {
    return d == D && (precision == DDMGNN_FP64 || tiles <= VT_MAX_FP32);
}

// Parts of one allocation, each on a cache line; a first pass without a base measures it.
struct Carver {
    char* base;
    size_t used = 0;
    template <typename T>
    T* take(size_t n) {
        T* p = base ? reinterpret_cast<T*>(base + used) : nullptr;
        used += (n * sizeof(T) + 255) / 256 * 256;
        return p;
    }
};

// Tiles of the sub-meshes of at most kMaxSubNodes nodes: their nodes by decreasing
// in-degree (tnode), so a tile's edge rows are its first node's in-degree (made even: rows
// are summed in pairs). The sub-meshes that the BF16 kernel does not run (need: its LDS
// bytes) come first: BF16 keeps arrays for those only. f(sub-mesh, first slot, position,
// edge rows) for every tile; rest: the tiles of those sub-meshes; returns all.
template <class F>
TileCount for_tiles(const HostSetup& hs, const std::vector<uint32_t>& need, TileCount& rest, F f) {
    TileCount n;
    for (int side = 0; side < 2; ++side) {
        for (int32_t i = 0; i < hs.K; ++i) {
            const int64_t b = hs.sub_ptr[i], k = hs.sub_ptr[i + 1] - b;
            if ((need[(size_t)i] <= MFMA_LDS_LIMIT) != (side == 1) || k > kMaxSubNodes) continue;
            for (int64_t q = 0; q < k; q += VT_TILE) {
                const int64_t slot = b + hs.tnode[b + q];
                const int64_t deg = (hs.edge_ptr[slot + 1] - hs.edge_ptr[slot] + 1) & ~int64_t(1);
                f(i, b, q, deg);
                ++n.tiles;
                n.rows += deg;
            }
        }
        if (side == 0) rest = n;
    }
    return n;
}
void list_tiles(ddmgnn_problem* P) {
    if (!P->vt_first.empty()) return;
    P->vt_first.assign((size_t)P->hs.K, 0);
    int64_t rows = 0;
    P->vt_all = for_tiles(P->hs, P->mfma_need, P->vt_rest, [&](int32_t i, int64_t b, int64_t q, int64_t deg) {
        if (q == 0) P->vt_first[i] = (int32_t)P->vt_tiles.size();
        P->vt_tiles.push_back(make_int4((int)b, (int)q, (int)rows, (int)deg));
        rows += deg;
    });
}

// The nodes of P's tiles and the slots' tile lanes (hook: a one-problem table to build
// with, left holding P).
hipError_t prepare_tile_nodes(ddmgnn_problem* P, DevBuf<DevProb>& hook) {
    hipStream_t s = P->ctx->stream;
    list_tiles(P);
    const size_t nt = P->vt_tiles.size(), K = (size_t)P->hs.K;
    const DevProb v = make_view(P);
    hipError_t e = launch_set_view(hook.p, v, s);
    if (e != hipSuccess || P->vt_pos) return e;
    // the tiles and the first of every sub-mesh: one copy
    std::vector<VtTile> host(P->vt_tiles);
    host.resize(nt + (K + 3) / 4);
    std::memcpy(host.data() + nt, P->vt_first.data(), K * sizeof(int32_t));
    auto carve = [&](Carver c, bool set) {
        VtTile* info = c.take<VtTile>(host.size());
        int2* node = c.take<int2>(nt * VT_TILE);
        int32_t* pos = c.take<int32_t>((size_t)P->hs.sk);
        if (set) {
            P->vt_info = info;
            P->vt_first_dev = reinterpret_cast<int32_t*>(info + nt);
            P->vt_node = node;
            P->vt_pos = pos;
        }
        return c.used;
    };
    e = P->vt_mem.alloc(carve(Carver{nullptr}, false));
    if (e == hipSuccess) e = upload_async(P->vt_mem.p, host.data(), host.size() * sizeof(VtTile), s);
    if (e != hipSuccess) return e;
    carve(Carver{P->vt_mem.p}, true);
    e = launch_vt_nodes(hook.p, P->vt_info, (int)nt, P->vt_node, P->vt_pos, s);
    if (e != hipSuccess)
        P->vt_pos = nullptr;  // a failed build is retried whole
    else
        P->device_bytes += tile_node_bytes((int64_t)nt, P->hs.sk, P->hs.K);
    return e;
}

// Frees P's tile arrays in one precision.
template <typename T>
void drop_tiles(ddmgnn_problem* P, VtBufs<T>& V) {
    if (V.mem.p) P->device_bytes -= tile_bytes(V.n, sizeof(T) == 8);
    V.mem.reset();
    V.v = VtVecs<T>{};
    V.n = TileCount{};
}

// P's FP64 / FP32 forward keeps one workgroup per sub-mesh from now on.
int make_untiled(ddmgnn_problem* P) {
    drop_tiles(P, P->vt64);
    drop_tiles(P, P->vt32);
    P->untiled = true;
    return DDMGNN_OK;
}

// Builds the arrays of P's tiled forward in type T for its first n.tiles tiles (hook: a
// one-problem table to build with); where they cannot be allocated P becomes untiled.
template <typename T>
int prepare_tiles(ddmgnn_problem* P, VtBufs<T>& V, const TileCount& n, DevBuf<DevProb>& hook, bool& changed) {
    if (V.mem.p && V.n.tiles >= n.tiles) return DDMGNN_OK;
    hipStream_t s = P->ctx->stream;
    const int64_t nt = n.tiles, rows = n.rows + VT_ROWS;
    if (nt * VT_TILE >= INT32_MAX) return make_untiled(P);  // tile lanes are 32-bit (edge records' offsets are not)
    hipError_t e = prepare_tile_nodes(P, hook);
    if (e == hipErrorOutOfMemory) return make_untiled(P);
    HIP_TRY(e);
    constexpr bool f64 = sizeof(T) == 8;
    const size_t er = (size_t)rows * VT_TILE, pad = (size_t)VT_ROWS * VT_TILE, qn = (size_t)(nt * VT_TILE + 1) * 2 * D;
    VtRec<T>* rec = nullptr;
    VtVecs<T> v{};
    auto carve = [&](Carver c) {
        rec = c.take<VtRec<T>>(er);
        v.info = f64 ? nullptr : c.take<T>((size_t)nt * VT_TILE * 4);
        v.h = c.take<T>((size_t)nt * 64 * 4);
        for (T*& q : v.q) q = c.take<T>(qn);
        v.rec = rec;
        return c.used;
    };
    drop_tiles(P, V);
    changed = true;
    DevBuf<char> mem;  // moved in last: a failed build is retried whole
    e = mem.alloc(carve(Carver{nullptr}));
    if (e == hipErrorOutOfMemory) return make_untiled(P);
    HIP_TRY(e);
    carve(Carver{mem.p});
    HIP_TRY(hipMemsetAsync(rec + er - pad, 0, pad * sizeof(VtRec<T>), s));
    const T inf = std::numeric_limits<T>::infinity();
    for (T* q : v.q) HIP_TRY(launch_vt_fill(q + qn - 2 * D, 2 * D, -inf, s));
    HIP_TRY(launch_vt_edges(hook.p, P->vt_info, (int)nt, P->vt_node, P->vt_pos,
                            f64 ? nullptr : reinterpret_cast<VtRec<float>*>(rec),
                            f64 ? reinterpret_cast<VtRec<double>*>(rec) : nullptr, s));
    std::swap(V.mem.p, mem.p);
    std::swap(V.mem.n, mem.n);
    V.v = v;
    V.n = n;
    P->device_bytes += tile_bytes(n, f64);
    return DDMGNN_OK;
}

int solo_batch(ddmgnn_problem* P);

// Training structures of a problem: per slot, its row of A_i = R_i A R_i^T
// (local columns, ascending), and per tile lane its edges in both directions (those it
// sends ordered by edge index).
int prepare_train(ddmgnn_problem* P) {
    if (P->lm_ptr.p) return DDMGNN_OK;
    hipStream_t s = P->ctx->stream;
    const auto& hs = P->hs;
    std::vector<int32_t> rowptr(hs.n + 1), col(hs.nnz), sub_nodes(hs.sk);
    std::vector<double> val(hs.nnz);
    HIP_TRY(hipMemcpyAsync(rowptr.data(), P->rowptr.p, rowptr.size() * 4, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(col.data(), P->col.p, col.size() * 4, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(val.data(), P->val.p, val.size() * 8, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(sub_nodes.data(), P->sub_nodes.p, sub_nodes.size() * 4, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    std::vector<int32_t> lm_ptr(hs.sk + 1, 0), oe_ptr(hs.sk + 1, 0), oe_edge(std::max<int64_t>(hs.n_edges, 1));
    std::vector<uint16_t> lm_col, oe_recv(std::max<int64_t>(hs.n_edges, 1));
    std::vector<float> lm_val;
    lm_col.reserve((size_t)hs.sk * 7);
    lm_val.reserve((size_t)hs.sk * 7);
    for (int32_t i = 0; i < hs.K; ++i) {
        const int64_t b = hs.sub_ptr[i], e = hs.sub_ptr[i + 1];
        const int32_t* first = sub_nodes.data() + b;
        const int32_t* last = sub_nodes.data() + e;
        for (int64_t q = b; q < e; ++q) {
            const int32_t j = sub_nodes[q];
            for (int32_t a = rowptr[j]; a < rowptr[j + 1]; ++a) {
                const int32_t* f = std::lower_bound(first, last, col[a]);
                if (f == last || *f != col[a]) continue;
                lm_col.push_back((uint16_t)(f - first));
                lm_val.push_back((float)val[a]);
            }
            lm_ptr[q + 1] = (int32_t)lm_col.size();
        }
        for (int64_t q = b; q < e; ++q)
            for (int64_t t = hs.edge_ptr[q]; t < hs.edge_ptr[q + 1]; ++t) oe_ptr[b + hs.edge_src[t] + 1]++;
    }
    if (lm_col.size() >= (size_t)INT32_MAX) return fail(DDMGNN_E_INVALID, "local matrices too large");
    for (int64_t q = 0; q < hs.sk; ++q) oe_ptr[q + 1] += oe_ptr[q];
    std::vector<int32_t> fill(oe_ptr.begin(), oe_ptr.end() - 1);
    for (int32_t i = 0; i < hs.K; ++i) {
        const int64_t b = hs.sub_ptr[i], e = hs.sub_ptr[i + 1];
        for (int64_t q = b; q < e; ++q)
            for (int64_t t = hs.edge_ptr[q]; t < hs.edge_ptr[q + 1]; ++t) {
                const int32_t at = fill[b + hs.edge_src[t]]++;
                oe_edge[at] = (int32_t)t;
                oe_recv[at] = (uint16_t)(q - b);
            }
    }
    // Tiles (dss_tile.h), their out-edge rows and the edge records of both directions.
    list_tiles(P);
    const size_t nt = P->vt_tiles.size();
    std::vector<int2> out_rows(nt);
    int64_t rows = 0;
    for (size_t t = 0; t < nt; ++t) {
        const VtTile f = P->vt_tiles[t];
        const int64_t k = hs.sub_ptr[hs.slot_sub[f.x] + 1] - f.x;
        int32_t deg = 0;
        for (int64_t q = f.y; q < std::min<int64_t>(k, f.y + VT_TILE); ++q) {
            const int64_t slot = f.x + hs.tnode[f.x + q];
            deg = std::max(deg, oe_ptr[slot + 1] - oe_ptr[slot]);
        }
        deg = (deg + 1) & ~1;  // rows are summed in pairs
        out_rows[t] = make_int2((int)rows, deg);
        rows += deg;
    }
    if (P->vt_all.tiles * VT_TILE >= INT32_MAX || rows + VT_ROWS >= INT32_MAX)
        return fail(DDMGNN_E_INVALID, "tile lanes or edge rows beyond 32 bits");
    if (int rc = solo_batch(P)) return rc;
    HIP_TRY(prepare_tile_nodes(P, P->solo->hook));
    std::vector<int32_t> map;
    std::vector<TrainEntry> ent;
    build_train_maps(map, ent);
    DevBuf<int32_t> oe_edge_d, oe_ptr_d;
    DevBuf<uint16_t> oe_recv_d;
    HIP_TRY(oe_ptr_d.upload(oe_ptr.data(), oe_ptr.size(), s));
    HIP_TRY(oe_edge_d.upload(oe_edge.data(), oe_edge.size(), s));
    HIP_TRY(oe_recv_d.upload(oe_recv.data(), oe_recv.size(), s));
    HIP_TRY(P->tr_map.upload(map.data(), map.size(), s));
    HIP_TRY(P->tr_ent.upload(ent.data(), ent.size(), s));
    HIP_TRY(P->tr_orows.upload(out_rows.data(), nt, s));
    const size_t ni = (size_t)(P->vt_all.rows + VT_ROWS) * VT_TILE, no = (size_t)(rows + VT_ROWS) * VT_TILE;
    HIP_TRY(P->tr_rin.alloc(ni));
    HIP_TRY(P->tr_rout.alloc(no));
    // the rows past the last tile are read, not looked at
    HIP_TRY(hipMemsetAsync(P->tr_rin.p, 0, ni * sizeof(TrainEdge), s));
    HIP_TRY(hipMemsetAsync(P->tr_rout.p, 0, no * sizeof(TrainEdge), s));
    const TrainEdgeArgs ea{P->vt_info, P->tr_orows.p, (int)nt, P->vt_node, P->vt_pos, P->edge_ptr.p,
                           P->edge_src.p, P->edge_nd.p, oe_ptr_d.p, oe_edge_d.p, oe_recv_d.p, P->xy64.p,
                           P->tr_rin.p, P->tr_rout.p};
    HIP_TRY(launch_train_edges(ea, s));
    HIP_TRY(P->lm_val.upload(lm_val.data(), lm_val.size(), s));
    HIP_TRY(P->lm_col.upload(lm_col.data(), lm_col.size(), s));
    HIP_TRY(hipStreamSynchronize(s));  // before the temporaries go
    P->tr_out_rows = std::move(out_rows);
    HIP_TRY(P->lm_ptr.upload(lm_ptr.data(), lm_ptr.size(), s));  // last: says that all is there
    P->device_bytes += lm_ptr.size() * 4 + lm_col.size() * 2 + lm_val.size() * 4 + map.size() * 4 +
                       ent.size() * sizeof(TrainEntry) + nt * sizeof(int2) + (ni + no) * sizeof(TrainEdge);
    return DDMGNN_OK;
}

int32_t sub_tiles(const ddmgnn_problem* P, int32_t i) {
    return (int32_t)((P->hs.sub_ptr[i + 1] - P->hs.sub_ptr[i] + VT_TILE - 1) / VT_TILE);
}

// The lists of a side that runs in tiles, for the problems' present forms.
int split_side(Batch& B, DssSide& S) {
    std::vector<uint8_t> now;
    for (const ddmgnn_problem* P : B.probs) now.push_back(P->untiled ? 1 : 0);
    if (S.untiled == now) return DDMGNN_OK;
    if (!S.untiled.empty()) {  // captured launches read the old lists
        B.graph.reset();
        B.brief.reset();
    }
    S.untiled.clear();
    std::vector<int2> subs, plain, order;
    S.max_k_plain = 0;
    for (const int2& w : S.host) {
        const ddmgnn_problem* P = B.probs[w.x];
        (now[w.x] ? plain : subs).push_back(w);
        if (now[w.x]) S.max_k_plain = std::max(S.max_k_plain, (int)(P->hs.sub_ptr[w.y + 1] - P->hs.sub_ptr[w.y]));
    }
    order = subs;
    std::sort(order.begin(), order.end(), [](const int2& a, const int2& b) { return a.x != b.x ? a.x < b.x : a.y < b.y; });
    std::vector<int4> v;
    for (const int2& w : order) {
        const ddmgnn_problem* P = B.probs[w.x];
        for (int32_t t = P->vt_first[w.y], e = t + sub_tiles(P, w.y); t < e; ++t)
            v.push_back(make_int4(w.x, t, P->vt_tiles[t].z, P->vt_tiles[t].w));
    }
    if (v.size() > (size_t)INT32_MAX) return fail(DDMGNN_E_INVALID, "too many tiles in one batch");
    if (int rc = upload_list(S.items, v, B.ctx->stream)) return rc;
    if (!plain.empty()) {
        if (int rc = upload_list(S.subs, subs, B.ctx->stream)) return rc;
        if (int rc = upload_list(S.plain, plain, B.ctx->stream)) return rc;
    }
    S.n_items = (int)v.size();
    S.n_subs = (int)subs.size();
    S.n_plain = (int)plain.size();
    S.untiled = now;
    return DDMGNN_OK;
}

// Allocates what the DSS launches of this precision need (fallback storage,
// LDS attributes). Not allowed during stream capture; returns true in
// `changed` when a problem's buffers moved (the table must be re-uploaded).
int prepare_dss(Batch& B, int precision, bool& changed) {
    changed = false;
    const bool bf16 = precision == DDMGNN_BF16;
    if (bf16 && B.n_mfma + B.n_mfma_small) HIP_TRY(prepare_dss_mfma(MFMA_LDS_LIMIT));
    const int valu_prec = bf16 ? DDMGNN_FP32 : precision;
    const bool f64 = valu_prec == DDMGNN_FP64;
    const int d = B.model->d;
    // sub-meshes beyond kMaxSubNodes: h, c and Q per slot in global memory
    for (ddmgnn_problem* P : B.probs) {
        if (!P->has_big) continue;
        const size_t sk = (size_t)P->hs.sk;
        if (f64 && P->qglobal64.n < sk * 2 * d) {
            HIP_TRY(P->qglobal64.alloc(sk * 2 * d));
            changed = true;
        }
        if (!f64 && P->qglobal32.n < sk * 2 * d) {
            HIP_TRY(P->qglobal32.alloc(sk * 2 * d));
            changed = true;
        }
        if (f64 && P->hglobal64.n < sk * d) {
            HIP_TRY(P->hglobal64.alloc(sk * d));
            changed = true;
        }
        if (!f64 && P->hglobal32.n < sk * d) {
            HIP_TRY(P->hglobal32.alloc(sk * d));
            changed = true;
        }
        if (P->cglobal.n < sk) {
            HIP_TRY(P->cglobal.alloc(sk));
            changed = true;
        }
    }
    DssSide& S = bf16 ? B.rest : B.valu;
    if (S.n == 0) return DDMGNN_OK;
    const bool tiled = runs_tiled(d, valu_prec, S.tiles);
    if (tiled) {
        for (ddmgnn_problem* P : B.probs) {
            if (P->untiled || (bf16 && !any_valu_bf16(P))) continue;
            list_tiles(P);
            const TileCount& n = bf16 ? P->vt_rest : P->vt_all;
            const int rc = f64 ? prepare_tiles(P, P->vt64, n, B.hook, changed) : prepare_tiles(P, P->vt32, n, B.hook, changed);
            if (rc) return rc;
        }
        if (int rc = split_side(B, S)) return rc;
        if (S.n_plain == 0) return DDMGNN_OK;
    }
    const bool in_lds = valu_q_in_lds(tiled ? S.max_k_plain : S.max_k, valu_prec, d);
    for (ddmgnn_problem* P : B.probs) {
        if ((bf16 && !any_valu_bf16(P)) || (tiled && !P->untiled)) continue;
        const size_t sk = (size_t)P->hs.sk;
        if (!in_lds) {
            if (f64 && P->qglobal64.n < sk * 2 * d) {
                HIP_TRY(P->qglobal64.alloc(sk * 2 * d));
                changed = true;
            }
            if (!f64 && P->qglobal32.n < sk * 2 * d) {
                HIP_TRY(P->qglobal32.alloc(sk * 2 * d));
                changed = true;
            }
        }
        if (f64 && P->hglobal64.n < sk * d) {
            HIP_TRY(P->hglobal64.alloc(sk * d));
            changed = true;
        }
    }
    if (in_lds) HIP_TRY(prepare_dss_valu(valu_prec, d, LDS_LIMIT - 1024));
    return DDMGNN_OK;
}

// The FP64 or FP32 forward of a side's sub-meshes.
int enqueue_side(Batch& B, const DssSide& S, const DevProb* tab, int precision, int apply, bool check) {
    hipStream_t s = B.ctx->launch;
    const ModelDev& M = *B.model;
    const int2* work = S.work.p;
    int n = S.n, max_k = S.max_k;
    if (runs_tiled(M.d, precision, S.tiles)) {
        const bool solo = B.probs.size() == 1;
        const int2* subs = S.n_plain ? S.subs.p : S.work.p;
        if (precision == DDMGNN_FP64)
            HIP_TRY(launch_dss_tiles<double>(tab, subs, S.n_subs, S.items.p, S.n_items, solo, M.kbar, M.alpha, apply,
                                             M.vt64.p, s, check));
        else
            HIP_TRY(launch_dss_tiles<float>(tab, subs, S.n_subs, S.items.p, S.n_items, solo, M.kbar, M.alpha, apply,
                                            M.vt32.p, s, check));
        work = S.plain.p;
        n = S.n_plain;
        max_k = S.max_k_plain;
    }
    const bool qlds = valu_q_in_lds(max_k, precision, M.d);
    HIP_TRY(launch_dss_valu(tab, work, n, precision, M.d, qlds, M.kbar, M.alpha, apply, M.theta32.p, M.theta64.p,
                            qlds ? valu_shmem(max_k, precision, M.d) : 0, s, check));
    return DDMGNN_OK;
}

// Local solves over every sub-mesh of the table: the DSS forward (apply:
// restriction and s r~), or the exact solves of DDM-LU.
int enqueue_dss(Batch& B, const DevProb* tab, int precision, int apply, bool capturing, int local = DDMGNN_LOCAL_GNN) {
    hipStream_t s = B.ctx->launch;
    const ModelDev& M = *B.model;
    const bool check = !capturing;
    if (local == DDMGNN_LOCAL_LU) {
        const LuWork w{B.lu_small.p, B.n_lu_small, B.valu.max_k, B.lu_big.p, B.n_lu_big, B.max_k_all,
                       B.lu_subs.p, B.n_lu_subs};
        HIP_TRY(launch_lu_local(tab, w, s, check));
        return DDMGNN_OK;
    }
    HIP_TRY(launch_dss_big(tab, B.work_big.p, B.n_big, precision == DDMGNN_BF16 ? DDMGNN_FP32 : precision, M.d,
                           M.kbar, M.alpha, apply, M.theta32.p, M.theta64.p, s, check));
    if (precision == DDMGNN_BF16) {
        DssMfmaArgs a{tab, B.work_mfma.p, M.steps.p, M.dec.p, M.kbar, (float)M.alpha, apply};
        if (B.n_mfma > 0 && B.n_mfma_small > 0) {
            // the two workgroup sizes on two streams, so that either launch's last
            // round overlaps the other's work; joined back before the next kernel
            ddmgnn_ctx* ctx = B.ctx;
            HIP_TRY(hipEventRecord(ctx->fork_ev, s));
            HIP_TRY(hipStreamWaitEvent(ctx->side, ctx->fork_ev, 0));
            DssMfmaArgs small = a;
            small.work = B.work_mfma_small.p;
            HIP_TRY(launch_dss_mfma(small, B.n_mfma_small, B.lds_mfma_small, MFMA_SMALL_BLOCK, ctx->side, check));
            HIP_TRY(hipEventRecord(ctx->join_ev, ctx->side));
            HIP_TRY(launch_dss_mfma(a, B.n_mfma, B.lds_mfma, MFMA_BLOCK, s, check));
            HIP_TRY(hipStreamWaitEvent(s, ctx->join_ev, 0));
        } else {
            HIP_TRY(launch_dss_mfma(a, B.n_mfma, B.lds_mfma, MFMA_BLOCK, s, check));
            a.work = B.work_mfma_small.p;
            HIP_TRY(launch_dss_mfma(a, B.n_mfma_small, B.lds_mfma_small, MFMA_SMALL_BLOCK, s, check));
        }
        return enqueue_side(B, B.rest, tab, DDMGNN_FP32, apply, check);
    }
    return enqueue_side(B, B.valu, tab, precision, apply, check);
}

IterArgs iter_args(const ddmgnn_solve_opts& o, int mode) {
    IterArgs ia{};
    ia.mode = mode;
    ia.m = mode == DDMGNN_FCG ? o.m_max : mode == DDMGNN_FGMRES ? o.restart : 1;
    ia.unweighted = o.prolong == DDMGNN_PROLONG_UNWEIGHTED;
    ia.coarse = o.coarse;
    return ia;
}

// One preconditioner apply z = M(r) over the table (mode < 0: no Krylov dots).
// ev (optional): events recorded after the DSS (ev[1]), coarse (ev[2]) and prolong (ev[3]) launches.
int enqueue_apply(Batch& B, const DevProb* tab, const ddmgnn_solve_opts& o, int mode, hipEvent_t* ev,
                  bool capturing) {
    if (int rc = enqueue_dss(B, tab, o.precision, 1, capturing, o.local_solver)) return rc;
    hipStream_t s = B.ctx->launch;
    if (ev) HIP_TRY(hipEventRecord(ev[1], s));
    if (o.coarse) HIP_TRY(launch_coarse(tab, B.coarse_rows.p, B.n_coarse, s, !capturing));
    if (ev) HIP_TRY(hipEventRecord(ev[2], s));
    HIP_TRY(launch_prolong(tab, B.vec_blk.p, B.n_vec, iter_args(o, mode), s, !capturing));
    if (ev) HIP_TRY(hipEventRecord(ev[3], s));
    return DDMGNN_OK;
}

// One FCG/PCG/CG iteration of every problem of the batch. ev: optional 5
// profiling events (before DSS, after DSS / coarse / prolong, end).
int enqueue_iteration(Batch& B, const ddmgnn_solve_opts& o, hipEvent_t* ev, bool capturing) {
    hipStream_t s = B.ctx->launch;
    const int mode = o.krylov;
    if (ev) HIP_TRY(hipEventRecord(ev[0], s));
    if (mode == DDMGNN_FGMRES) {
        HIP_TRY(launch_fgmres_next(B.tab.p, B.vec_blk.p, B.n_vec, iter_args(o, mode), s, !capturing));
        if (int rc = enqueue_apply(B, B.tab.p, o, mode, ev, capturing)) return rc;
        HIP_TRY(launch_fgmres_step(B.tab.p, B.vec_blk.p, B.n_vec, (int)B.probs.size(), iter_args(o, mode), s,
                                   !capturing));
        if (ev) HIP_TRY(hipEventRecord(ev[4], s));
        return DDMGNN_OK;
    }
    if (mode == DDMGNN_CG) {
        if (ev)
            for (int q = 1; q < 4; ++q) HIP_TRY(hipEventRecord(ev[q], s));
    } else {
        if (int rc = enqueue_apply(B, B.tab.p, o, mode, ev, capturing)) return rc;
    }
    HIP_TRY(launch_krylov(B.tab.p, B.vec_blk.p, B.n_vec, (int)B.probs.size(), iter_args(o, mode), s, !capturing));
    if (ev) HIP_TRY(hipEventRecord(ev[4], s));
    return DDMGNN_OK;
}

uint64_t graph_key(const ddmgnn_solve_opts& o, int count) {
    const int m = o.krylov == DDMGNN_FGMRES ? o.restart : o.m_max;
    return ((uint64_t)o.local_solver << 56) | ((uint64_t)o.krylov << 52) | ((uint64_t)(m & 0xff) << 44) |
           ((uint64_t)o.precision << 40) | ((uint64_t)o.prolong << 38) | ((uint64_t)(o.coarse != 0) << 36) |
           (uint64_t)(uint32_t)count;
}

// Iterations of a solve's captured graph. A tiled forward is a launch per block, so an iteration
// after the last one, in which every kernel returns at once, costs some 50 us, and capturing
// one 40. A solve whose batch's last one took at most two graphs of four (or the first)
// therefore replays such a graph, its flags read after 4, 8, 16 and then every check_every
// of them; a longer one's successor has the whole chunk as one graph, which saves 1%. FP32
// solves of two iterations, with chunks of 16 and now: 5k nodes 1,200 and 530 us, the first on
// its problem 2,110 and 910 (one workgroup per sub-mesh: 1,170 and 1,480); 300 nodes 1,175 and
// 510, 2,050 and 850 (845 and 1,115).
constexpr int BRIEF_CHUNK = 4;
int brief_chunk(const Batch& B, const ddmgnn_solve_opts& o) {
    const int check = std::max(1, o.check_every);
    if (o.krylov == DDMGNN_CG || o.local_solver == DDMGNN_LOCAL_LU || B.last_it > 2 * BRIEF_CHUNK) return check;
    const bool bf16 = o.precision == DDMGNN_BF16;
    const DssSide& S = bf16 ? B.rest : B.valu;
    const bool tiled = S.n > 0 && runs_tiled(B.model->d, bf16 ? DDMGNN_FP32 : o.precision, S.tiles);
    return tiled ? std::min(check, BRIEF_CHUNK) : check;
}

// Captures `count` iterations of the batch into G, unless it holds them (on the context's own
// stream: the caller's stream may be the null stream, which cannot be captured).
int capture_chunk(Batch& B, Batch::Graph& G, const ddmgnn_solve_opts& o, int count) {
    ddmgnn_ctx* ctx = B.ctx;
    if (G.exec && G.key == graph_key(o, count)) return DDMGNN_OK;
    G.reset();
    hipGraph_t g = nullptr;
    HIP_TRY(hipStreamBeginCapture(ctx->cap, hipStreamCaptureModeRelaxed));
    ctx->launch = ctx->cap;
    int crc = 0;
    for (int c = 0; c < count && crc == 0; ++c) crc = enqueue_iteration(B, o, nullptr, true);
    ctx->launch = ctx->stream;
    hipError_t ce = hipStreamEndCapture(ctx->cap, &g);
    if (crc || ce != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        hipStreamCaptureStatus cst = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(ctx->cap, &cst) == hipSuccess && cst != hipStreamCaptureStatusNone) {
            hipGraph_t g2 = nullptr;
            (void)hipStreamEndCapture(ctx->cap, &g2);
            if (g2) (void)hipGraphDestroy(g2);
        }
        if (crc) return crc;
        HIP_TRY(ce);
    }
    HIP_TRY(hipGetLastError());
    hipError_t ie = hipGraphInstantiate(&G.exec, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (ie != hipSuccess) G.exec = nullptr;
    HIP_TRY(ie);
    G.key = graph_key(o, count);
    return DDMGNN_OK;
}

int upload_table(Batch& B) {
    B.views.resize(B.probs.size());
    for (size_t i = 0; i < B.probs.size(); ++i) B.views[i] = make_view(B.probs[i]);
    return upload_list(B.tab, B.views, B.ctx->stream);
}

// Workgroup list and problem list of the problems flagged in `which`.
int upload_subset(Batch& B, const std::vector<uint8_t>* which) {
    std::vector<int2> sub;
    std::vector<int> list;
    for (size_t i = 0; i < B.probs.size(); ++i) {
        if (which && !(*which)[i]) continue;
        list.push_back((int)i);
        const int nb = problem_vec_blocks(B.probs[i]);
        for (int b = 0; b < nb; ++b) sub.push_back(make_int2((int)i, b));
    }
    B.n_sub_blk = (int)sub.size();
    B.n_sub_list = (int)list.size();
    if (int rc = upload_list(B.sub_list, list, B.ctx->stream)) return rc;
    return upload_list(B.sub_blk, sub, B.ctx->stream);
}

int solo_batch(ddmgnn_problem* P) {
    if (P->solo) return DDMGNN_OK;
    ddmgnn_problem* one[1] = {P};
    return build_batch(P->ctx, one, 1, P->solo);
}

// Solve every problem of the batch from its u0 with options o.
int solve_batch(ddmgnn_ctx* ctx, Batch& B, const ddmgnn_solve_opts& o, double* const* u_out, ddmgnn_stats* stats) {
    hipStream_t s = ctx->stream;
    const int nb = (int)B.probs.size();
    for (ddmgnn_problem* P : B.probs) {
        P->rtol = o.rtol;
        P->max_it = o.max_it;
    }
    hipEvent_t ev0, ev1;
    HIP_TRY(hipEventCreate(&ev0));
    HIP_TRY(hipEventCreate(&ev1));
    struct EvGuard {
        hipEvent_t a, b;
        std::vector<hipEvent_t> v;
        ~EvGuard() {
            (void)hipEventDestroy(a);
            (void)hipEventDestroy(b);
            for (auto e : v) (void)hipEventDestroy(e);
        }
    } guard{ev0, ev1, {}};
    if (int rc = batch_begin(B, o, nullptr)) return rc;
    HIP_TRY(hipEventRecord(ev0, s));
    HIP_TRY(launch_init(B.tab.p, B.vec_blk.p, B.n_vec, nullptr, nb, s));
    // Iterations between host polls of the converged flags; a captured chunk
    // is replayed as a whole (problems that finish inside it idle).
    const int check = std::max(1, o.check_every);
    const bool use_graph = o.graph && !o.profile;
    const int brief = brief_chunk(B, o);
    if (o.profile) {
        guard.v.resize((size_t)check * 5);
        for (auto& e : guard.v) HIP_TRY(hipEventCreate(&e));
    }
    double t_dss = 0, t_coarse = 0, t_prolong = 0, t_krylov = 0;
    int n_dss = 0, it = 0, it_seen = 0;
    bool done = o.max_it <= 0;
    while (!done) {
        int n_chunk = use_graph ? check : std::min(check, o.max_it - it);
        if (use_graph && brief < check) {
            if (int rc = capture_chunk(B, B.brief, o, brief)) return rc;
            const int replays = std::max(1, std::min(it, check) / brief);  // up to 4, 8, 16, ... iterations
            for (int q = 0; q < replays; ++q) HIP_TRY(hipGraphLaunch(B.brief.exec, s));
            n_chunk = replays * brief;
        } else if (use_graph) {
            if (int rc = capture_chunk(B, B.graph, o, check)) return rc;
            HIP_TRY(hipGraphLaunch(B.graph.exec, s));
        } else {
            for (int c = 0; c < n_chunk; ++c)
                if (int rc = enqueue_iteration(B, o, o.profile ? &guard.v[(size_t)c * 5] : nullptr, false)) return rc;
        }
        if (int rc = batch_poll(B)) return rc;
        it += n_chunk;
        bool all = true;
        int max_it_done = 0;
        for (int i = 0; i < nb; ++i) {
            all = all && B.host_st[i].done;
            max_it_done = std::max(max_it_done, B.host_st[i].it);
        }
        done = all || it >= o.max_it;
        if (o.profile) {
            // iterations it_seen .. max_it_done-1 did work; later ones exited at once
            const int worked = std::min(n_chunk, std::max(0, max_it_done - it_seen));
            for (int c = 0; c < worked; ++c) {
                hipEvent_t* ev = &guard.v[(size_t)c * 5];
                float a = 0, b = 0, cc = 0, d = 0;
                HIP_TRY(hipEventElapsedTime(&a, ev[0], ev[1]));
                HIP_TRY(hipEventElapsedTime(&b, ev[1], ev[2]));
                HIP_TRY(hipEventElapsedTime(&cc, ev[2], ev[3]));
                HIP_TRY(hipEventElapsedTime(&d, ev[3], ev[4]));
                t_dss += a;
                t_coarse += b;
                t_prolong += cc;
                t_krylov += d;
                if (o.krylov != DDMGNN_CG) ++n_dss;
            }
        }
        it_seen = max_it_done;
    }
    B.last_it = it_seen;
    HIP_TRY(hipEventRecord(ev1, s));
    if (int rc = batch_true_residual(B, nullptr)) return rc;
    for (int i = 0; i < nb; ++i)
        HIP_TRY(hipMemcpyAsync(u_out[i], B.probs[i]->u.p, B.probs[i]->hs.n * sizeof(double),
                               hipMemcpyDeviceToDevice, s));
    HIP_TRY(hipStreamSynchronize(s));
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, ev0, ev1));
    int first_bad = DDMGNN_OK;
    for (int i = 0; i < nb; ++i) {
        const KState& k = B.host_st[i];
        const bool converged = k.status == 0 && k.rel <= o.rtol;
        if (stats) {
            ddmgnn_stats& S = stats[i];
            std::memset(&S, 0, sizeof(S));
            S.iterations = k.it;
            S.converged = converged;
            S.rel_residual = k.rel;
            S.true_rel_residual = k.r0n > 0 ? std::sqrt(k.rr_true) / k.r0n : 0.0;
            S.solve_ms = ms;
            S.dss_launches = n_dss;
            S.dss_ms = t_dss;
            S.coarse_ms = t_coarse;
            S.prolong_ms = t_prolong;
            S.krylov_ms = t_krylov;
            S.dss_kernel = dss_kernel_of(B.probs[i], o);
            S.status = k.status ? k.status : (converged ? DDMGNN_OK : DDMGNN_E_MAXIT);
            S.latency_ms = ms;
        }
        if (first_bad == DDMGNN_OK) {
            if (k.status) first_bad = fail(k.status, "Krylov breakdown or non-finite residual");
            else if (!converged) first_bad = fail(DDMGNN_E_MAXIT, "not converged within max_it");
        }
    }
    return first_bad;
}

}  // namespace

// ------------------------------------------------------------------ batch API
void BatchDeleter::operator()(Batch* b) const { delete b; }

int build_batch(ddmgnn_ctx* ctx, ddmgnn_problem* const* probs, int n, BatchPtr& out) {
    BatchPtr B(new Batch());
    B->ctx = ctx;
    B->probs.assign(probs, probs + n);
    for (int i = 0; i < n; ++i) B->ids.push_back(probs[i]->id);
    B->model = probs[0]->model;
    struct W {
        int k, p, sub;
    };
    std::vector<W> all;
    std::vector<int2> vec, rows;
    for (int i = 0; i < n; ++i) {
        const ddmgnn_problem* P = probs[i];
        const auto& sp = P->hs.sub_ptr;
        for (int j = 0; j < P->hs.K; ++j) all.push_back({(int)(sp[j + 1] - sp[j]), i, j});
        const int nb = problem_vec_blocks(P);
        for (int b = 0; b < nb; ++b) vec.push_back(make_int2(i, b));
        for (int r = 0; r < P->hs.K; ++r) rows.push_back(make_int2(i, r));
    }
    // Largest sub-meshes first (a deterministic order: size, then problem, then sub-mesh).
    std::stable_sort(all.begin(), all.end(), [](const W& a, const W& b) {
        if (a.k != b.k) return a.k > b.k;
        if (a.p != b.p) return a.p < b.p;
        return a.sub < b.sub;
    });
    std::vector<int2> wm, wms, wb;
    auto add = [](DssSide& S, const W& w) {
        S.host.push_back(make_int2(w.p, w.sub));
        S.max_k = std::max(S.max_k, w.k);
        S.tiles += (w.k + VT_TILE - 1) / VT_TILE;
    };
    size_t lds_sb = 0, lds_db = 0, lds_small_sb = 0, lds_small_db = 0;
    for (const W& w : all) {
        B->all.push_back(make_int2(w.p, w.sub));
        B->max_k_all = std::max(B->max_k_all, w.k);
        const ddmgnn_problem* Q = probs[w.p];
        if (w.k > kMaxSubNodes) {
            wb.push_back(make_int2(w.p, w.sub));
            continue;
        }
        add(B->valu, w);
        if (mfma_runs_sub(Q, w.sub)) {
            const size_t need = Q->mfma_need[w.sub];
            // Each launch reserves the largest need of its members; with two Q'
            // buffers where they fit that reserve (up to the kernel's limit, or
            // half a compute unit's LDS for the small workgroups), one otherwise.
            const size_t need_db = Q->mfma_need_db[w.sub];
            if (w.k <= MFMA_SMALL_K && need <= (size_t)Q->tune.small_lds) {
                wms.push_back(make_int2(w.p, w.sub));
                lds_small_sb = std::max(lds_small_sb, need);
                if (need_db <= MFMA_SMALL_LDS) lds_small_db = std::max(lds_small_db, need_db);
            } else {
                wm.push_back(make_int2(w.p, w.sub));
                lds_sb = std::max(lds_sb, need);
                if (need_db <= MFMA_LDS_LIMIT) lds_db = std::max(lds_db, need_db);
            }
        } else {
            add(B->rest, w);
        }
    }
    B->lds_mfma = std::max(lds_sb, lds_db);
    B->lds_mfma_small = std::max(lds_small_sb, lds_small_db);
    hipStream_t s = ctx->stream;
    if (int rc = upload_list(B->work_mfma, wm, s)) return rc;
    if (int rc = upload_list(B->work_mfma_small, wms, s)) return rc;
    for (DssSide* S : {&B->valu, &B->rest}) {
        if (int rc = upload_list(S->work, S->host, s)) return rc;
        S->n = (int)S->host.size();
    }
    if (int rc = upload_list(B->work_big, wb, s)) return rc;
    if (int rc = upload_list(B->vec_blk, vec, s)) return rc;
    if (int rc = upload_list(B->coarse_rows, rows, s)) return rc;
    B->n_mfma = (int)wm.size();
    B->n_mfma_small = (int)wms.size();
    B->n_big = (int)wb.size();
    B->n_vec = (int)vec.size();
    B->n_coarse = (int)rows.size();
    HIP_TRY(B->st_gather.alloc(n));
    HIP_TRY(B->hook.alloc(1));
    HIP_TRY(hipHostMalloc((void**)&B->host_st, sizeof(KState) * n, hipHostMallocDefault));
    std::memset(B->host_st, 0, sizeof(KState) * n);
    if (int rc = upload_table(*B)) return rc;
    out = std::move(B);
    return DDMGNN_OK;
}

int batch_begin(Batch& B, const ddmgnn_solve_opts& o, const std::vector<uint8_t>* init) {
    bool changed = false;
    if (o.krylov != DDMGNN_CG && o.local_solver == DDMGNN_LOCAL_LU) {
        if (int rc = prepare_exact(B, changed)) return rc;
    } else if (o.krylov != DDMGNN_CG) {
        if (int rc = prepare_dss(B, o.precision, changed)) return rc;
    }
    if (o.krylov == DDMGNN_FGMRES)
        if (int rc = prepare_fgmres(B, o.restart, changed)) return rc;
    if (changed) {  // captured launches point at moved buffers
        B.graph.reset();
        B.brief.reset();
    }
    if (int rc = upload_table(B)) return rc;
    if (init) {
        if (int rc = upload_subset(B, init)) return rc;
        if (B.n_sub_blk)
            HIP_TRY(launch_init(B.tab.p, B.sub_blk.p, B.n_sub_blk, B.sub_list.p, B.n_sub_list, B.ctx->stream));
    }
    return DDMGNN_OK;
}

int batch_iterate(Batch& B, const ddmgnn_solve_opts& o, int count, bool use_graph) {
    if (use_graph) {
        if (int rc = capture_chunk(B, B.graph, o, count)) return rc;
        HIP_TRY(hipGraphLaunch(B.graph.exec, B.ctx->stream));
        return DDMGNN_OK;
    }
    for (int c = 0; c < count; ++c)
        if (int rc = enqueue_iteration(B, o, nullptr, false)) return rc;
    return DDMGNN_OK;
}

int batch_poll(Batch& B) {
    hipStream_t s = B.ctx->stream;
    const int n = (int)B.probs.size();
    HIP_TRY(launch_gather_states(B.tab.p, n, B.st_gather.p, s));
    HIP_TRY(hipMemcpyAsync(B.host_st, B.st_gather.p, sizeof(KState) * n, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    return DDMGNN_OK;
}

const KState& batch_state(const Batch& B, int i) { return B.host_st[i]; }
int batch_size(const Batch& B) { return (int)B.probs.size(); }
ddmgnn_problem* batch_problem(const Batch& B, int i) { return B.probs[i]; }

int batch_true_residual(Batch& B, const std::vector<uint8_t>* which) {
    if (which) {
        if (int rc = upload_subset(B, which)) return rc;
        if (B.n_sub_blk)
            HIP_TRY(launch_resid(B.tab.p, B.sub_blk.p, B.n_sub_blk, B.sub_list.p, B.n_sub_list, B.ctx->stream));
    } else {
        HIP_TRY(launch_resid(B.tab.p, B.vec_blk.p, B.n_vec, nullptr, (int)B.probs.size(), B.ctx->stream));
    }
    return batch_poll(B);
}

int host_desc(const ddmgnn_problem_desc* in, HostDesc& h, const ddmgnn_problem_desc** out) {
    if (in->mem_kind == DDMGNN_MEM_HOST) {
        *out = in;
        return DDMGNN_OK;
    }
    if (in->mem_kind != DDMGNN_MEM_DEVICE) return fail(DDMGNN_E_INVALID, "mem_kind must be HOST or DEVICE");
    const int64_t n = in->n_nodes, nt = in->n_tri, K = in->n_sub;
    if (n <= 0 || nt <= 0 || K <= 0 || !in->a_rowptr || !in->sub_ptr)
        return fail(DDMGNN_E_INVALID, "empty problem");
    auto get = [&](auto& vec, const auto* src, int64_t count) -> hipError_t {
        if (!src || count <= 0) return hipSuccess;
        vec.resize((size_t)count);
        return hipMemcpy(vec.data(), src, (size_t)count * sizeof(vec[0]), hipMemcpyDeviceToHost);
    };
    HIP_TRY(get(h.a_rowptr, in->a_rowptr, n + 1));
    HIP_TRY(get(h.sub_ptr, in->sub_ptr, K + 1));
    const int64_t nnz = h.a_rowptr[n], sk = h.sub_ptr[K];
    if (nnz < 0 || sk < 0) return fail(DDMGNN_E_INVALID, "negative sizes");
    HIP_TRY(get(h.xy, in->xy, 2 * n));
    HIP_TRY(get(h.tri, in->tri, 3 * nt));
    HIP_TRY(get(h.dirichlet, in->dirichlet, n));
    HIP_TRY(get(h.a_col, in->a_col, nnz));
    HIP_TRY(get(h.a_val, in->a_val, nnz));
    HIP_TRY(get(h.b, in->b, n));
    HIP_TRY(get(h.u0, in->u0, n));
    HIP_TRY(get(h.sub_nodes, in->sub_nodes, sk));
    HIP_TRY(get(h.weights, in->weights, sk));
    auto ptr = [](auto& vec) { return vec.empty() ? nullptr : vec.data(); };
    ddmgnn_problem_desc& d = h.desc;
    d = *in;
    d.mem_kind = DDMGNN_MEM_HOST;
    d.xy = ptr(h.xy);
    d.tri = ptr(h.tri);
    d.dirichlet = ptr(h.dirichlet);
    d.a_rowptr = ptr(h.a_rowptr);
    d.a_col = ptr(h.a_col);
    d.a_val = ptr(h.a_val);
    d.b = ptr(h.b);
    d.u0 = ptr(h.u0);
    d.sub_ptr = ptr(h.sub_ptr);
    d.sub_nodes = ptr(h.sub_nodes);
    d.weights = ptr(h.weights);
    *out = &h.desc;
    return DDMGNN_OK;
}

int problem_vec_blocks(const ddmgnn_problem* P) {
    const int autom = vec_blocks(P->hs.n);
    return P->tune.vec_blocks > 0 ? std::min(autom, P->tune.vec_blocks) : autom;
}

// FGMRES storage for cycles of R steps: basis (R + 1) x n, Z R x n, partial sums
// (R + 1) x VEC_GRID, small arrays (H, rotations, g, y, tmp).
size_t fgmres_bytes(int64_t n, int R) {
    return 8 * ((size_t)(2 * R + 1) * n + (size_t)(R + 1) * VEC_GRID + (size_t)R * R + 6 * R + 2);
}

int dss_kernel_of(const ddmgnn_problem* P, const ddmgnn_solve_opts& o) {
    if (o.local_solver == DDMGNN_LOCAL_LU) return 3;
    if (o.precision == DDMGNN_FP64) return 0;
    if (o.precision != DDMGNN_BF16 || all_valu_bf16(P)) return 1;
    return any_valu_bf16(P) ? 4 : 2;
}

int check_opts(const ddmgnn_solve_opts& o) {
    if (o.krylov < 0 || o.krylov > 3) return fail(DDMGNN_E_INVALID, "krylov must be FCG, PCG, CG or FGMRES");
    if (o.krylov == DDMGNN_FGMRES && (o.restart < 1 || o.restart > MAX_RESTART))
        return fail(DDMGNN_E_INVALID, "restart must be in [1, 64]");
    if (o.krylov == DDMGNN_FCG && (o.m_max < 1 || o.m_max > MAX_M)) return fail(DDMGNN_E_INVALID, "m_max must be in [1, 4]");
    if (!(o.rtol >= 0.0)) return fail(DDMGNN_E_INVALID, "rtol must be >= 0");
    if (o.max_it < 0) return fail(DDMGNN_E_INVALID, "max_it must be >= 0");
    if (o.precision < 0 || o.precision > 2) return fail(DDMGNN_E_INVALID, "precision must be FP64, FP32 or BF16");
    if (o.prolong < 0 || o.prolong > 1) return fail(DDMGNN_E_INVALID, "prolong must be POU or UNWEIGHTED");
    if (o.local_solver < 0 || o.local_solver > 1) return fail(DDMGNN_E_INVALID, "local_solver must be GNN or LU");
    return DDMGNN_OK;
}

// Bytes a problem counts for its exact local solves: a square per sub-mesh, which is what
// the small ones hold and covers the tiles (about half), the partial products and most of
// the panels of the factorisation of the others.
size_t lu_bytes(const HostSetup& hs) {
    size_t b = 0;
    for (int32_t i = 0; i < hs.K; ++i) {
        const int64_t k = hs.sub_ptr[i + 1] - hs.sub_ptr[i];
        b += (size_t)(k * lu_ld(k)) * 8 + 8;
    }
    return b;
}

// Bytes of the nodes of a problem's tiles, and of the tiled forward's arrays in one precision.
size_t tile_node_bytes(int64_t tiles, int64_t sk, int32_t K) {
    return (size_t)tiles * (sizeof(VtTile) + VT_TILE * sizeof(int2)) + 4 * ((size_t)sk + K);
}
size_t tile_bytes(const TileCount& n, bool f64) {
    const size_t e = f64 ? 8 : 4;
    return (size_t)n.tiles * ((f64 ? 0 : 16 * VT_TILE) + 256 * e) + (size_t)(n.rows + VT_ROWS) * VT_TILE * 2 * e +
           (size_t)(n.tiles * VT_TILE + 1) * 4 * D * e;
}

// Bytes of what the forward of a model of width d allocates for a problem (prepare_dss), in
// tiles where it runs them or not; hs after prepare_upload.
size_t forward_bytes(const HostSetup& hs, int d, int precision, bool tiles) {
    const bool bf16 = precision == DDMGNN_BF16, f64 = precision == DDMGNN_FP64;
    const size_t e = f64 ? 8 : 4, sk = (size_t)hs.sk;
    bool q = hs.has_big, h = hs.has_big;  // of every slot: sender rows, states
    int max_k = 0;
    for (int32_t i = 0; i < hs.K; ++i) {
        const int k = (int)(hs.sub_ptr[i + 1] - hs.sub_ptr[i]);
        if (k <= kMaxSubNodes && !(bf16 && d <= D && hs.mfma_need[i] <= MFMA_LDS_LIMIT)) max_k = std::max(max_k, k);
    }
    size_t b = hs.has_big ? 8 * sk : 0;
    if (max_k > 0) {
        TileCount rest;
        const TileCount all = for_tiles(hs, hs.mfma_need, rest, [](int32_t, int64_t, int64_t, int64_t) {});
        const TileCount& n = bf16 ? rest : all;
        if (tiles && runs_tiled(d, f64 ? DDMGNN_FP64 : DDMGNN_FP32, n.tiles)) {
            b += tile_node_bytes(all.tiles, hs.sk, hs.K) + tile_bytes(n, f64);
        } else {
            q = q || !valu_q_in_lds(max_k, f64 ? DDMGNN_FP64 : DDMGNN_FP32, d);
            h = h || f64;
        }
    }
    return b + (q ? sk * 2 * d * e : 0) + (h ? sk * d * e : 0);
}

// Bytes of the coarse level's scratch beyond the direction ring (create_problem).
size_t coarse_scratch_bytes(int64_t n, int32_t K) {
    const size_t need = coarse_scratch_doubles(K);
    return (size_t)2 * (MAX_M + 1) * n < need ? 8 * need : 0;
}

size_t problem_device_bytes(int64_t n, int64_t nnz, int32_t K, int64_t sk, int64_t ne) {
    size_t b = 0;
    b += 4 * (n + 1) + 12 * nnz;                 // CSR
    b += 8 * n * 2 + n;                          // b, u0, dirichlet
    b += 4 * (K + 1) + 12 * sk;                  // sub_ptr, sub_nodes, weights
    b += 4 * (sk + 1) + (2 + 4) * (ne + 8);      // edge_ptr, edge_src, edge_nd
    b += 4 * (ne + sk * (MFMA_EC - 1)) + 4 * (K + 1);  // padded edge records (bound), their ranges
    b += 16 * sk + 16 * sk + 8 * sk;             // tiles, xy64, xyc32
    b += 4 * (n + 1) + 8 * sk;                   // node_ptr, node_slots, slot_sub
    b += 8 * (size_t)K * K + 24 * (size_t)K;     // a0inv, s, y0, y
    b += 8 * sk;                                 // local
    b += 8 * n * (3 + 2 * (MAX_M + 1));          // u, r, z, direction ring
    b += 8 * N_PART * VEC_GRID + 16 + sizeof(KState);
    return b;
}

// The device-ready host arrays of a problem (HostSetup::upload_ready): plain
// host work, run by the caller of create_problem or by a server's setup worker.
std::string prepare_upload(const ddmgnn_problem_desc& desc, HostSetup& hs) {
    if (hs.upload_ready) return "";
    const int64_t n = hs.n, sk = hs.sk;
    const int K = hs.K;
    constexpr int64_t CH = 1 << 16;  // elements per task of the conversion loops
    hs.sp32.resize((size_t)K + 1);
    for (int i = 0; i <= K; ++i) hs.sp32[i] = (int32_t)desc.sub_ptr[i];
    hs.ep32.resize((size_t)sk + 1);
    hs.np32.resize((size_t)n + 1);
    hs.xy64.resize((size_t)2 * sk);
    hs.xyc32.resize((size_t)2 * sk);
    parallel_for((sk + CH) / CH, [&](int64_t c) {
        for (int64_t k = c * CH; k < std::min(sk + 1, (c + 1) * CH); ++k) hs.ep32[k] = (int32_t)hs.edge_ptr[k];
        for (int64_t k = c * CH; k < std::min(sk, (c + 1) * CH); ++k) {
            const int32_t v = desc.sub_nodes[k];
            hs.xy64[2 * k] = desc.xy[2 * v];
            hs.xy64[2 * k + 1] = desc.xy[2 * v + 1];
            hs.xyc32[2 * k] = (float)hs.xyc[2 * k];
            hs.xyc32[2 * k + 1] = (float)hs.xyc[2 * k + 1];
        }
    });
    parallel_for((n + CH) / CH, [&](int64_t c) {
        for (int64_t i = c * CH; i < std::min(n + 1, (c + 1) * CH); ++i) hs.np32[i] = (int32_t)hs.node_ptr[i];
    });
    // padded by 8 entries: the chunked edge loops read up to 3 past a node's last edge
    hs.src_pad.assign(hs.edge_src.begin(), hs.edge_src.end());
    hs.src_pad.resize(hs.src_pad.size() + 8, 0);
    hs.nd_pad.assign(hs.edge_nd.begin(), hs.edge_nd.end());
    hs.nd_pad.resize(hs.nd_pad.size() + 8, 0.0f);
    // MFMA kernel records, per tile of MFMA_TILE nodes (tile order): slot-major
    // [slot][lane] blocks padded with sentinel records (sender k_i, |d| 0)
    // to the tile's largest in-degree rounded up to MFMA_EC. Tile records
    // hold the block's offset in the sub-mesh (low 24 bits) and its number
    // of MFMA_EC-slot chunks (high 8 bits). Sub-meshes are independent: the
    // sizes of their edge blocks first, then their records in parallel.
    hs.mfma_need.assign(K, 0);
    hs.mfma_need_db.assign(K, 0);
    std::vector<int64_t> esize((size_t)K, 0);
    std::atomic<int> too_big{0};
    parallel_for(K, [&](int64_t i) {
        const int64_t b = desc.sub_ptr[i], k = desc.sub_ptr[i + 1] - b;
        if (k > kMaxSubNodes) return;  // the VALU kernel's global-memory form runs it: no tile records
        int64_t size = 0;
        for (int64_t t0 = 0; t0 < k; t0 += MFMA_TILE) {
            int maxdeg = 0;
            for (int64_t q = t0; q < std::min<int64_t>(k, t0 + MFMA_TILE); ++q) {
                const int64_t slot = b + hs.tnode[b + q];
                maxdeg = std::max<int>(maxdeg, (int)(hs.edge_ptr[slot + 1] - hs.edge_ptr[slot]));
            }
            const int nch = (maxdeg + MFMA_EC - 1) / MFMA_EC;
            if (nch > 255 || size + (int64_t)nch * MFMA_EC * MFMA_TILE >= (1 << 24)) too_big = 1;
            size += (int64_t)nch * MFMA_EC * MFMA_TILE;
        }
        esize[i] = size;
    });
    if (too_big) return "sub-mesh edge block too large for the MFMA tile records";
    std::vector<int32_t>& epad = hs.mfma_epad;
    epad.assign((size_t)K + 1, 0);
    for (int i = 0; i < K; ++i) {
        if (epad[i] + esize[i] >= INT32_MAX) return "edge records beyond 32-bit offsets";
        epad[i + 1] = (int32_t)(epad[i] + esize[i]);
    }
    std::vector<uint32_t>& er = hs.mfma_erec;
    er.assign((size_t)epad[K], 0u);
    hs.has_big = false;
    std::vector<TileNode> tiles(sk);
    parallel_for(K, [&](int64_t i) {
        const int64_t b = desc.sub_ptr[i], e = desc.sub_ptr[i + 1];
        const int k = (int)(e - b);
        if (k > kMaxSubNodes) {
            hs.mfma_need[i] = UINT32_MAX;
            hs.mfma_need_db[i] = UINT32_MAX;
            return;
        }
        std::vector<int64_t> cand;  // per lane of a tile: its in-edges, in order
        std::vector<uint8_t> taken;
        size_t off = 0;
        for (int t0 = 0; t0 < k; t0 += MFMA_TILE) {
            const int t1 = std::min(k, t0 + MFMA_TILE);
            int maxdeg = 0;
            for (int q = t0; q < t1; ++q) {
                const int64_t slot = b + hs.tnode[b + q];
                maxdeg = std::max<int>(maxdeg, (int)(hs.edge_ptr[slot + 1] - hs.edge_ptr[slot]));
            }
            const int nch = (maxdeg + MFMA_EC - 1) / MFMA_EC;
            uint32_t* blk = er.data() + epad[i] + off;
            std::fill(blk, blk + (size_t)nch * MFMA_EC * MFMA_TILE, mfma_edge_record(k, 0));
            // Slot by slot, each lane takes the first remaining in-edge whose sender
            // row starts on the least used LDS bank of the slot (rows are 5 dwords
            // apart), so a wavefront's gathers spread over the banks. This only
            // reorders each node's message sum.
            cand.assign((size_t)(t1 - t0) * maxdeg, -1);
            taken.assign(cand.size(), 0);
            for (int q = t0; q < t1; ++q) {
                const int64_t slot = b + hs.tnode[b + q];
                for (int64_t t = hs.edge_ptr[slot]; t < hs.edge_ptr[slot + 1]; ++t)
                    cand[(size_t)(q - t0) * maxdeg + (t - hs.edge_ptr[slot])] = t;
            }
            for (int w = 0; w < maxdeg; ++w) {
                int used[32] = {0};
                for (int q = t0; q < t1; ++q) {
                    const int64_t* c = cand.data() + (size_t)(q - t0) * maxdeg;
                    uint8_t* tk = taken.data() + (size_t)(q - t0) * maxdeg;
                    int best = -1;
                    for (int x = 0; x < maxdeg && c[x] >= 0; ++x)
                        if (!tk[x] && (best < 0 || used[(5 * hs.edge_src[c[x]]) % 32] <
                                                       used[(5 * hs.edge_src[c[best]]) % 32]))
                            best = x;
                    if (best < 0) continue;
                    const int64_t t = c[best];
                    tk[best] = 1;
                    used[(5 * hs.edge_src[t]) % 32]++;
                    blk[(size_t)w * MFMA_TILE + (q - t0)] = mfma_edge_record(hs.edge_src[t], (uint16_t)(hs.erec[t] >> 16));
                }
            }
            for (int q = t0; q < t1; ++q) {
                const int32_t j = hs.tnode[b + q];
                const int64_t slot = b + j;
                TileNode& tn = tiles[b + q];
                tn.e0 = (int32_t)((uint32_t)off | ((uint32_t)nch << 24));
                tn.j = (uint16_t)j;
                tn.deg = (uint16_t)(hs.edge_ptr[slot + 1] - hs.edge_ptr[slot]);
                tn.xh = hs.xyhl[4 * slot + 0];
                tn.xl = hs.xyhl[4 * slot + 1];
                tn.yh = hs.xyhl[4 * slot + 2];
                tn.yl = hs.xyhl[4 * slot + 3];
            }
            off += (size_t)nch * MFMA_EC * MFMA_TILE;
        }
        hs.mfma_need[i] = (uint32_t)mfma_lds_need(k, esize[i]);
        hs.mfma_need_db[i] = (uint32_t)mfma_lds_need(k, esize[i], true);
    });
    for (int i = 0; i < K; ++i) hs.has_big = hs.has_big || hs.mfma_need[i] == UINT32_MAX;
    static_assert(sizeof(TileNode) == 4 * sizeof(uint32_t), "tile records are four words");
    hs.mfma_tiles.resize((size_t)4 * sk);
    if (sk) std::memcpy(hs.mfma_tiles.data(), tiles.data(), (size_t)sk * sizeof(TileNode));
    hs.upload_ready = true;
    return "";
}

int create_problem(ddmgnn_ctx* ctx, const ddmgnn_problem_desc& desc, std::shared_ptr<ModelDev> model,
                   HostSetup&& hs_in, ddmgnn_problem** out, hipStream_t stream) {
    auto P = std::make_unique<ddmgnn_problem>();
    P->ctx = ctx;
    P->id = g_next_id.fetch_add(1);
    P->hs = std::move(hs_in);
    P->model = std::move(model);
    {
        const std::string e = prepare_upload(desc, P->hs);
        if (!e.empty()) return fail(DDMGNN_E_INVALID, e);
    }
    const auto& hs = P->hs;
    const int64_t n = hs.n, sk = hs.sk;
    const int K = hs.K;
    hipStream_t s = stream ? stream : ctx->stream;
    HIP_TRY(P->rowptr.upload(desc.a_rowptr, n + 1, s));
    HIP_TRY(P->col.upload(desc.a_col, hs.nnz, s));
    HIP_TRY(P->val.upload(desc.a_val, hs.nnz, s));
    HIP_TRY(P->b.upload(desc.b, n, s));
    HIP_TRY(P->u0.upload(desc.u0, n, s));
    HIP_TRY(P->dirichlet.upload(desc.dirichlet, n, s));
    HIP_TRY(P->sub_ptr.upload(hs.sp32.data(), K + 1, s));
    HIP_TRY(P->sub_nodes.upload(desc.sub_nodes, sk, s));
    HIP_TRY(P->weights.upload(desc.weights, sk, s));
    HIP_TRY(P->edge_ptr.upload(hs.ep32.data(), sk + 1, s));
    HIP_TRY(P->edge_src.upload(hs.src_pad.data(), hs.src_pad.size(), s));
    HIP_TRY(P->node_ptr.upload(hs.np32.data(), n + 1, s));
    HIP_TRY(P->node_slots.upload(hs.node_slots.data(), sk, s));
    HIP_TRY(P->slot_sub.upload(hs.slot_sub.data(), sk, s));
    HIP_TRY(P->xy64.upload(hs.xy64.data(), 2 * sk, s));
    HIP_TRY(P->xyc32.upload(hs.xyc32.data(), 2 * sk, s));
    // Krylov vectors; the direction ring also serves the coarse setup below as scratch
    HIP_TRY(P->ring.alloc((size_t)2 * (MAX_M + 1) * n));
    if (!hs.a0inv.empty()) {
        HIP_TRY(P->a0inv.upload(hs.a0inv.data(), (size_t)K * K, s));
    } else {  // the coarse operator and its inverse, formed on the device
        const size_t need = coarse_scratch_doubles(K);
        HIP_TRY(P->a0inv.alloc((size_t)K * K));
        HIP_TRY(P->coarse_diag0.alloc((size_t)K));
        HIP_TRY(P->coarse_status.alloc(1));
        if (P->ring.n < need) HIP_TRY(P->coarse_scratch.alloc(need));
        HIP_TRY(hipMemsetAsync(P->coarse_status.p, 0, sizeof(int), s));
        HIP_TRY(launch_coarse_assemble(P->rowptr.p, P->col.p, P->val.p, P->sub_ptr.p, P->sub_nodes.p, P->weights.p,
                                       P->node_ptr.p, P->node_slots.p, P->slot_sub.p, K, P->a0inv.p,
                                       P->coarse_diag0.p, s));
        HIP_TRY(launch_coarse_invert(P->a0inv.p, K, P->coarse_diag0.p,
                                     P->coarse_scratch.p ? P->coarse_scratch.p : P->ring.p, P->coarse_status.p, s));
        const int rc = pivots_ok(P->coarse_status, s);
        if (rc == DDMGNN_E_NOT_SPD) return fail(rc, "coarse matrix R_0 A R_0^T is not positive definite");
        if (rc) return rc;
    }
    P->mfma_need = hs.mfma_need;
    P->mfma_need_db = hs.mfma_need_db;
    P->has_big = hs.has_big;
    HIP_TRY(P->tiles.upload(reinterpret_cast<const TileNode*>(hs.mfma_tiles.data()), (size_t)sk, s));
    HIP_TRY(P->erec.upload(hs.mfma_erec.data(), std::max<size_t>(hs.mfma_erec.size(), 1), s));
    HIP_TRY(P->epad_sub.upload(hs.mfma_epad.data(), hs.mfma_epad.size(), s));
    HIP_TRY(P->edge_nd.upload(hs.nd_pad.data(), hs.nd_pad.size(), s));
    HIP_TRY(P->s.alloc(K));
    HIP_TRY(P->y0.alloc(K));
    HIP_TRY(P->y.alloc(K));
    HIP_TRY(P->local.alloc(sk));
    HIP_TRY(P->u.alloc(n));
    HIP_TRY(P->r.alloc(n));
    HIP_TRY(P->z.alloc(n));
    HIP_TRY(P->st.alloc(1));
    HIP_TRY(P->partials.alloc((size_t)N_PART * VEC_GRID));
    HIP_TRY(hipMemsetAsync(P->st.p, 0, sizeof(KState), s));
    HIP_TRY(hipStreamSynchronize(s));
    P->device_bytes = problem_device_bytes(n, hs.nnz, K, sk, hs.n_edges) + P->coarse_scratch.n * sizeof(double);
    // host copies of the uploaded arrays are not needed again
    HostSetup& h = P->hs;
    std::vector<int32_t>().swap(h.sp32);
    std::vector<int32_t>().swap(h.ep32);
    std::vector<int32_t>().swap(h.np32);
    std::vector<double>().swap(h.xy64);
    std::vector<float>().swap(h.xyc32);
    std::vector<float>().swap(h.nd_pad);
    std::vector<uint16_t>().swap(h.src_pad);
    std::vector<uint32_t>().swap(h.mfma_erec);
    std::vector<uint32_t>().swap(h.mfma_tiles);
    std::vector<int32_t>().swap(h.mfma_epad);
    h.upload_ready = false;
    *out = P.release();
    return DDMGNN_OK;
}

}  // namespace ddmgnn

using namespace ddmgnn;

ddmgnn_ctx::~ddmgnn_ctx() {
    last_batch.reset();
    if (host_pinned) (void)hipHostFree(host_pinned);
    if (cap) (void)hipStreamDestroy(cap);
    if (side) (void)hipStreamDestroy(side);
    if (fork_ev) (void)hipEventDestroy(fork_ev);
    if (join_ev) (void)hipEventDestroy(join_ev);
}

// Drops the cached batches that hold P (its own and the context's last one).
void drop_batches(ddmgnn_problem* P) {
    P->solo.reset();
    if (P->ctx && P->ctx->last_batch) {
        const auto& B = *P->ctx->last_batch;
        if (std::find(B.ids.begin(), B.ids.end(), P->id) != B.ids.end()) P->ctx->last_batch.reset();
    }
}

ddmgnn_problem::~ddmgnn_problem() { drop_batches(this); }

// ------------------------------------------------------------------ C ABI
extern "C" {

const char* ddmgnn_last_error(void) { return g_err.c_str(); }
const char* ddmgnn_version(void) { return "ddmgnn 0.2 gfx950"; }
int32_t ddmgnn_max_subdomain_nodes(void) { return kMaxSubNodesAny; }

void ddmgnn_default_opts(ddmgnn_solve_opts* o) {
    o->krylov = DDMGNN_FCG;
    o->m_max = 1;
    o->rtol = 1e-6;
    o->max_it = 10000;
    o->precision = DDMGNN_FP32;
    o->prolong = DDMGNN_PROLONG_POU;
    o->coarse = 1;
    o->check_every = 16;
    o->profile = 0;
    o->graph = 1;
    o->local_solver = DDMGNN_LOCAL_GNN;
    o->restart = 30;
}

int ddmgnn_ctx_create(void* hip_stream, ddmgnn_ctx** out) {
    if (!out) return fail(DDMGNN_E_INVALID, "null output pointer");
    auto c = std::make_unique<ddmgnn_ctx>();
    c->stream = (hipStream_t)hip_stream;
    c->launch = c->stream;
    HIP_TRY(hipGetDevice(&c->device));
    HIP_TRY(hipStreamCreateWithFlags(&c->cap, hipStreamNonBlocking));
    HIP_TRY(hipStreamCreateWithFlags(&c->side, hipStreamNonBlocking));
    HIP_TRY(hipEventCreateWithFlags(&c->fork_ev, hipEventDisableTiming));
    HIP_TRY(hipEventCreateWithFlags(&c->join_ev, hipEventDisableTiming));
    HIP_TRY(c->partials.alloc(VEC_GRID));
    HIP_TRY(c->scalar.alloc(1));
    HIP_TRY(hipHostMalloc((void**)&c->host_pinned, 256, hipHostMallocDefault));
    HIP_TRY(noalloc_init(c->device));  // with the context's device current
    *out = c.release();
    return DDMGNN_OK;
}

int ddmgnn_ctx_destroy(ddmgnn_ctx* ctx) {
    delete ctx;
    return DDMGNN_OK;
}

int ddmgnn_model_create(ddmgnn_ctx* ctx, const ddmgnn_model_desc* desc, const float* theta, int64_t n_theta,
                        ddmgnn_model** out) {
    if (!ctx || !desc || !theta || !out) return fail(DDMGNN_E_INVALID, "null argument");
    const int d = desc->d;
    if (d != 5 && d != 10 && d != 20) return fail(DDMGNN_E_INVALID, "latent width d must be 5, 10 or 20");
    if (desc->kbar < 1) return fail(DDMGNN_E_INVALID, "kbar must be >= 1");
    const int64_t expect = (int64_t)desc->kbar * (11 * d * d + 15 * d + 1);
    if (n_theta != expect) return fail(DDMGNN_E_INVALID, "n_theta must equal kbar*(11d^2+15d+1)");
    for (int64_t i = 0; i < n_theta; ++i)
        if (!std::isfinite(theta[i])) return fail(DDMGNN_E_INVALID, "non-finite weight");
    auto m = std::make_unique<ddmgnn_model>();
    m->kbar = desc->kbar;
    m->d = desc->d;
    m->alpha = desc->alpha;
    m->theta.assign(theta, theta + n_theta);
    std::vector<MfmaStep> steps;
    std::vector<MfmaDec> dec;
    if (d == D) {
        build_mfma_blobs(m->theta.data(), m->kbar, steps, dec);
    } else if (d < D) {  // the matrix-core kernel runs the model embedded in width 10
        std::vector<float> padded;
        pad_theta_to_d10(m->theta.data(), m->kbar, d, padded);
        build_mfma_blobs(padded.data(), m->kbar, steps, dec);
    }
    auto dev = std::make_shared<ModelDev>();
    dev->id = g_next_id.fetch_add(1);
    dev->kbar = m->kbar;
    dev->d = d;
    dev->mfma = d <= D;
    dev->alpha = m->alpha;
    hipStream_t s = ctx->stream;
    std::vector<double> th64(m->theta.begin(), m->theta.end());
    HIP_TRY(dev->theta32.upload(m->theta.data(), m->theta.size(), s));
    HIP_TRY(dev->theta64.upload(th64.data(), th64.size(), s));
    HIP_TRY(dev->steps.upload(steps.data(), steps.size(), s));
    HIP_TRY(dev->dec.upload(dec.data(), dec.size(), s));
    // (last: with the tiles' blobs before theta32 the one-workgroup FP32 kernel, whose scalar loads
    // of the weights are its longest chain, takes 3,235 us instead of 3,160 at 1M nodes)
    if (d == D) {
        std::vector<double> b64;
        std::vector<float> b32;
        build_vt_blobs(m->theta.data(), m->kbar, b64, b32);
        HIP_TRY(dev->vt64.upload(b64.data(), b64.size(), s));
        HIP_TRY(dev->vt32.upload(b32.data(), b32.size(), s));
    }
    m->dev = std::move(dev);
    *out = m.release();
    return DDMGNN_OK;
}

int ddmgnn_model_init_xavier(const ddmgnn_model_desc* desc, uint64_t seed, float* theta, int64_t n_theta) {
    if (!desc || !theta) return fail(DDMGNN_E_INVALID, "null argument");
    const int64_t d = desc->d, kbar = desc->kbar;
    if (d < 1 || kbar < 1 || n_theta != kbar * (11 * d * d + 15 * d + 1))
        return fail(DDMGNN_E_INVALID, "n_theta must equal kbar*(11d^2+15d+1)");
    uint64_t state = seed;
    auto next = [&]() {  // splitmix64
        state += 0x9E3779B97F4A7C15ull;
        uint64_t z = state;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    };
    int64_t pos = 0;
    auto layer = [&](int64_t fan_out, int64_t fan_in) {
        const double a = std::sqrt(6.0 / (double)(fan_in + fan_out));
        for (int64_t i = 0; i < fan_out * fan_in; ++i) {
            const double u = (double)(next() >> 11) * 0x1.0p-53;
            theta[pos++] = (float)(a * (2.0 * u - 1.0));
        }
        for (int64_t i = 0; i < fan_out; ++i) theta[pos++] = 0.0f;
    };
    for (int64_t k = 0; k < kbar; ++k) {
        for (int phi = 0; phi < 2; ++phi) {
            layer(d, 2 * d + 3);
            layer(d, d);
        }
        layer(d, 3 * d + 1);
        layer(d, d);
        layer(d, d);
        layer(1, d);
    }
    return DDMGNN_OK;
}

int ddmgnn_model_destroy(ddmgnn_model* m) {
    delete m;
    return DDMGNN_OK;
}

int ddmgnn_validate_problem(const ddmgnn_problem_desc* desc_in) {
    if (!desc_in) return fail(DDMGNN_E_INVALID, "null descriptor");
    HostDesc hd;
    const ddmgnn_problem_desc* desc = nullptr;
    if (int rc = host_desc(desc_in, hd, &desc)) return rc;
    std::string e = validate(*desc);
    if (!e.empty()) return fail(DDMGNN_E_INVALID, e);
    return DDMGNN_OK;
}

int ddmgnn_problem_create(ddmgnn_ctx* ctx, const ddmgnn_problem_desc* desc_in, const ddmgnn_model* model,
                          ddmgnn_problem** out) {
    if (!ctx || !desc_in || !model || !out) return fail(DDMGNN_E_INVALID, "null argument");
    HostDesc hd;
    const ddmgnn_problem_desc* desc = nullptr;
    if (int rc = host_desc(desc_in, hd, &desc)) return rc;
    int rc = ddmgnn_validate_problem(desc);
    if (rc) return rc;
    HostSetup hs;
    std::string e = build_setup(*desc, hs, false);  // the coarse level is formed on the device
    if (!e.empty()) return fail(DDMGNN_E_INVALID, e);
    return create_problem(ctx, *desc, model->dev, std::move(hs), out);
}

int ddmgnn_problem_destroy(ddmgnn_problem* P) {
    delete P;
    return DDMGNN_OK;
}

int ddmgnn_problem_sizes(const ddmgnn_problem* P, int64_t* n, int64_t* nnz, int32_t* k, int64_t* sum_k,
                         int64_t* n_edges) {
    if (!P) return fail(DDMGNN_E_INVALID, "null problem");
    if (n) *n = P->hs.n;
    if (nnz) *nnz = P->hs.nnz;
    if (k) *k = P->hs.K;
    if (sum_k) *sum_k = P->hs.sk;
    if (n_edges) *n_edges = P->hs.n_edges;
    return DDMGNN_OK;
}

int ddmgnn_problem_set_tuning(ddmgnn_problem* P, const ddmgnn_tuning* t) {
    if (!P || !t) return fail(DDMGNN_E_INVALID, "null argument");
    if (t->small_lds < 0 || t->small_lds > (int32_t)MFMA_SMALL_LDS)
        return fail(DDMGNN_E_INVALID, "small_lds must be in [0, 80 KiB - 1 KiB]");
    if (t->vec_blocks != 0 && (t->vec_blocks < N_XCD || t->vec_blocks > VEC_GRID || t->vec_blocks % N_XCD))
        return fail(DDMGNN_E_INVALID, "vec_blocks must be 0 or a multiple of 8 in [8, 1024]");
    if (t->small_lds != P->tune.small_lds || t->vec_blocks != P->tune.vec_blocks) {
        P->tune = *t;
        drop_batches(P);
    }
    return DDMGNN_OK;
}

int ddmgnn_problem_get_tuning(const ddmgnn_problem* P, ddmgnn_tuning* t) {
    if (!P || !t) return fail(DDMGNN_E_INVALID, "null argument");
    *t = P->tune;
    return DDMGNN_OK;
}

int ddmgnn_autotune(ddmgnn_ctx* ctx, ddmgnn_problem* P, const ddmgnn_solve_opts* opts, int32_t iterations,
                    ddmgnn_tuning* best, double* ms_per_iteration) {
    if (!ctx || !P || !opts) return fail(DDMGNN_E_INVALID, "null argument");
    if (iterations < 1) return fail(DDMGNN_E_INVALID, "iterations must be >= 1");
    if (int rc = check_opts(*opts)) return rc;
    ddmgnn_solve_opts o = *opts;
    o.max_it = iterations;
    o.rtol = 0.0;  // run the capped number of iterations
    o.graph = 1;
    o.profile = 0;
    o.check_every = std::min(iterations, 16);
    // time per iteration of a candidate: best of two capped solves (the first of a
    // schedule also captures its graph)
    auto timed = [&](const ddmgnn_tuning& t, double& ms) -> int {
        if (int rc = ddmgnn_problem_set_tuning(P, &t)) return rc;
        if (int rc = solo_batch(P)) return rc;
        double best_ms = 1e300;
        for (int rep = 0; rep < 3; ++rep) {
            ddmgnn_stats st{};
            double* outs[1] = {P->z.p};  // the solution copy lands in scratch
            const int rc = solve_batch(ctx, *P->solo, o, outs, &st);
            if (rc && rc != DDMGNN_E_MAXIT) return rc;
            if (rep > 0) best_ms = std::min(best_ms, st.solve_ms / std::max(1, st.iterations));
        }
        ms = best_ms;
        return DDMGNN_OK;
    };
    const bool mfma = o.krylov != DDMGNN_CG && o.local_solver == DDMGNN_LOCAL_GNN &&
                      dss_kernel_of(P, o) == 2;
    ddmgnn_tuning cur{0, 0}, top{0, 0};
    double top_ms = 1e300;
    std::vector<int32_t> lds = {0};
    if (mfma) lds = {0, 48 * 1024, 64 * 1024, (int32_t)MFMA_SMALL_LDS};
    for (int32_t v : lds) {
        cur.small_lds = v;
        double ms = 0;
        if (int rc = timed(cur, ms)) return rc;
        if (ms < top_ms) {
            top_ms = ms;
            top = cur;
        }
    }
    cur = top;
    for (int32_t vb : {256, 512, 1024}) {
        if (vb > vec_blocks(P->hs.n)) continue;
        cur.vec_blocks = vb;
        double ms = 0;
        if (int rc = timed(cur, ms)) return rc;
        if (ms < top_ms) {
            top_ms = ms;
            top = cur;
        }
    }
    if (int rc = ddmgnn_problem_set_tuning(P, &top)) return rc;
    if (best) *best = top;
    if (ms_per_iteration) *ms_per_iteration = top_ms;
    return DDMGNN_OK;
}

int ddmgnn_problem_device_bytes(const ddmgnn_problem* P, int64_t* bytes) {
    if (!P || !bytes) return fail(DDMGNN_E_INVALID, "null argument");
    *bytes = (int64_t)P->device_bytes;
    return DDMGNN_OK;
}

int ddmgnn_setup_local_graph(const ddmgnn_problem_desc* desc_in, int32_t sub, int32_t* rowptr, int32_t* col,
                             int64_t* n_edges_sub) {
    if (!desc_in) return fail(DDMGNN_E_INVALID, "null descriptor");
    HostDesc hd;
    const ddmgnn_problem_desc* desc = nullptr;
    if (int rc = host_desc(desc_in, hd, &desc)) return rc;
    int rc = ddmgnn_validate_problem(desc);
    if (rc) return rc;
    if (sub < 0 || sub >= desc->n_sub) return fail(DDMGNN_E_INVALID, "sub-mesh index out of range");
    HostSetup hs;
    build_local_graphs(*desc, hs);
    const int64_t b = desc->sub_ptr[sub], e = desc->sub_ptr[sub + 1];
    const int64_t e0 = hs.edge_ptr[b], e1 = hs.edge_ptr[e];
    if (n_edges_sub) *n_edges_sub = e1 - e0;
    if (rowptr)
        for (int64_t k = b; k <= e; ++k) rowptr[k - b] = (int32_t)(hs.edge_ptr[k] - e0);
    if (col)
        for (int64_t q = e0; q < e1; ++q) col[q - e0] = hs.edge_src[q];
    return DDMGNN_OK;
}

int ddmgnn_setup_coarse(const ddmgnn_problem_desc* desc_in, double* a0, double* a0inv) {
    if (!desc_in) return fail(DDMGNN_E_INVALID, "null descriptor");
    HostDesc hd;
    const ddmgnn_problem_desc* desc = nullptr;
    if (int rc = host_desc(desc_in, hd, &desc)) return rc;
    int rc = ddmgnn_validate_problem(desc);
    if (rc) return rc;
    HostSetup hs;
    std::string e = build_setup(*desc, hs);
    if (!hs.a0.empty() && a0) std::memcpy(a0, hs.a0.data(), hs.a0.size() * sizeof(double));
    if (e == "NOT_SPD") return fail(DDMGNN_E_NOT_SPD, "coarse matrix R_0 A R_0^T is not positive definite");
    if (!e.empty()) return fail(DDMGNN_E_INVALID, e);
    if (a0inv) std::memcpy(a0inv, hs.a0inv.data(), hs.a0inv.size() * sizeof(double));
    return DDMGNN_OK;
}

int ddmgnn_setup_local_inverse(const ddmgnn_problem_desc* desc_in, int32_t sub, double* inv) {
    if (!desc_in) return fail(DDMGNN_E_INVALID, "null descriptor");
    HostDesc hd;
    const ddmgnn_problem_desc* desc = nullptr;
    if (int rc = host_desc(desc_in, hd, &desc)) return rc;
    int rc = ddmgnn_validate_problem(desc);
    if (rc) return rc;
    if (sub < 0 || sub >= desc->n_sub || !inv) return fail(DDMGNN_E_INVALID, "sub-mesh index out of range or null output");
    std::vector<double> m;
    if (!local_inverse(*desc, sub, m, true).empty())
        return fail(DDMGNN_E_NOT_SPD, "local matrix R_i A R_i^T is not positive definite");
    std::memcpy(inv, m.data(), m.size() * sizeof(double));
    return DDMGNN_OK;
}

int ddmgnn_spmv(ddmgnn_ctx* ctx, ddmgnn_problem* P, const double* x, double* y) {
    if (!ctx || !P || !x || !y) return fail(DDMGNN_E_INVALID, "null argument");
    HIP_TRY(launch_spmv(P->rowptr.p, P->col.p, P->val.p, x, y, (int)P->hs.n, problem_vec_blocks(P), ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    return DDMGNN_OK;
}

int ddmgnn_dot(ddmgnn_ctx* ctx, int64_t n, const double* x, const double* y, double* out) {
    if (!ctx || !out || n < 0 || n > INT32_MAX || (n > 0 && (!x || !y))) return fail(DDMGNN_E_INVALID, "invalid argument");
    if (n == 0) {
        *out = 0.0;
        return DDMGNN_OK;
    }
    HIP_TRY(launch_dot(x, y, (int)n, ctx->partials.p, ctx->scalar.p, ctx->stream, true));
    HIP_TRY(hipMemcpyAsync(ctx->host_pinned, ctx->scalar.p, sizeof(double), hipMemcpyDeviceToHost, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    *out = ctx->host_pinned[0];
    return DDMGNN_OK;
}

int ddmgnn_dot_noalloc(ddmgnn_ctx* ctx, int64_t n, const double* x, const double* y, double* out) {
    if (!ctx || !out || n < 0 || (n > 0 && (!x || !y))) return fail(DDMGNN_E_INVALID, "null argument or n < 0");
    if (n > DDMGNN_NOALLOC_DOT_MAX_N)
        return fail(DDMGNN_E_INVALID, "ddmgnn_dot_noalloc: n exceeds DDMGNN_NOALLOC_DOT_MAX_N (2^31 - 1)");
    double* scr = noalloc_scratch(ctx->device);
    if (!scr) return fail(DDMGNN_E_INVALID, "ddmgnn_dot_noalloc: no scratch address for the context's device");
    // n = 0 runs the same kernels over no rows: the partials are 0 and so is *out.
    HIP_TRY(launch_dot(x, y, (int)n, scr, out, ctx->stream, true));
    return DDMGNN_OK;
}

int ddmgnn_dss_forward(ddmgnn_ctx* ctx, ddmgnn_problem* P, int32_t precision, const double* c, double* out) {
    if (!ctx || !P || !c || !out) return fail(DDMGNN_E_INVALID, "null argument");
    if (precision < 0 || precision > 2) return fail(DDMGNN_E_INVALID, "bad precision");
    if (int rc = solo_batch(P)) return rc;
    Batch& B = *P->solo;
    bool changed = false;
    if (int rc = prepare_dss(B, precision, changed)) return rc;
    DevProb v = make_view(P);
    v.c_in = c;
    v.local = out;
    v.st = nullptr;
    HIP_TRY(launch_set_view(B.hook.p, v, ctx->stream));
    if (int rc = enqueue_dss(B, B.hook.p, precision, 0, false)) return rc;
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    return DDMGNN_OK;
}

int ddmgnn_dss_forward_sub(ddmgnn_ctx* ctx, ddmgnn_problem* P, int32_t precision, int32_t sub, const double* c,
                           double* out) {
    if (!ctx || !P || !c || !out) return fail(DDMGNN_E_INVALID, "null argument");
    if (precision < 0 || precision > 2) return fail(DDMGNN_E_INVALID, "bad precision");
    if (sub < 0 || sub >= P->hs.K) return fail(DDMGNN_E_INVALID, "sub-mesh index out of range");
    if (int rc = solo_batch(P)) return rc;
    Batch& B = *P->solo;
    bool changed = false;
    if (int rc = prepare_dss(B, precision, changed)) return rc;
    hipStream_t s = ctx->stream;
    const int64_t base = P->hs.sub_ptr[sub], k = P->hs.sub_ptr[sub + 1] - base;
    if (!P->one_work.p) {  // the last of them: a failed build is retried whole
        HIP_TRY(P->fwd_in.alloc((size_t)P->hs.sk));
        HIP_TRY(P->fwd_out.alloc((size_t)P->hs.sk));
        HIP_TRY(P->one_work.alloc(1));
    }
    const int2 item = make_int2(0, sub);
    HIP_TRY(upload_async(P->one_work.p, &item, sizeof(item), s));
    HIP_TRY(hipMemcpyAsync(P->fwd_in.p + base, c, (size_t)k * sizeof(double), hipMemcpyDeviceToDevice, s));
    DevProb v = make_view(P);
    v.c_in = P->fwd_in.p;
    v.local = P->fwd_out.p;
    v.st = nullptr;
    HIP_TRY(launch_set_view(B.hook.p, v, s));
    const ModelDev& M = *B.model;
    const int vprec = precision == DDMGNN_BF16 ? DDMGNN_FP32 : precision;
    const DssSide& S = precision == DDMGNN_BF16 ? B.rest : B.valu;
    if (k > kMaxSubNodes) {
        HIP_TRY(launch_dss_big(B.hook.p, P->one_work.p, 1, vprec, M.d, M.kbar, M.alpha, 0, M.theta32.p,
                               M.theta64.p, s, true));
    } else if (precision == DDMGNN_BF16 && mfma_runs_sub(P, sub)) {
        DssMfmaArgs a{B.hook.p, P->one_work.p, M.steps.p, M.dec.p, M.kbar, (float)M.alpha, 0};
        const size_t shmem = P->mfma_need_db[sub] <= MFMA_LDS_LIMIT ? P->mfma_need_db[sub] : P->mfma_need[sub];
        HIP_TRY(launch_dss_mfma(a, 1, shmem, MFMA_BLOCK, s, true));
    } else if (runs_tiled(M.d, vprec, S.tiles) && !P->untiled) {  // as prepare_dss
        std::vector<int4> tl;
        for (int32_t t = P->vt_first[sub], e = t + sub_tiles(P, sub); t < e; ++t)
            tl.push_back(make_int4(0, t, P->vt_tiles[t].z, P->vt_tiles[t].w));
        if (int rc = upload_list(P->one_tiles, tl, s)) return rc;
        if (vprec == DDMGNN_FP64)
            HIP_TRY(launch_dss_tiles<double>(B.hook.p, P->one_work.p, 1, P->one_tiles.p, (int)tl.size(), true, M.kbar,
                                             M.alpha, 0, M.vt64.p, s, true));
        else
            HIP_TRY(launch_dss_tiles<float>(B.hook.p, P->one_work.p, 1, P->one_tiles.p, (int)tl.size(), true, M.kbar,
                                            M.alpha, 0, M.vt32.p, s, true));
    } else {
        const bool qlds = valu_q_in_lds(S.max_k, vprec, M.d);  // as prepare_dss sized it
        HIP_TRY(launch_dss_valu(B.hook.p, P->one_work.p, 1, vprec, M.d, qlds, M.kbar, M.alpha, 0, M.theta32.p,
                                M.theta64.p, qlds ? valu_shmem(S.max_k, vprec, M.d) : 0, s, true));
    }
    HIP_TRY(hipMemcpyAsync(out, P->fwd_out.p + base, (size_t)k * sizeof(double), hipMemcpyDeviceToDevice, s));
    HIP_TRY(hipStreamSynchronize(s));
    return DDMGNN_OK;
}

int ddmgnn_time_apply_stages(ddmgnn_ctx* ctx, ddmgnn_problem* P, const ddmgnn_solve_opts* opts, const double* r,
                             double* z, int32_t reps, double* local_ms, double* coarse_ms, double* glue_ms) {
    if (!ctx || !P || !opts || !r || !z) return fail(DDMGNN_E_INVALID, "null argument");
    if (r == z) return fail(DDMGNN_E_INVALID, "r and z must not alias");
    if (reps < 1) return fail(DDMGNN_E_INVALID, "reps must be >= 1");
    if (int rc = check_opts(*opts)) return rc;
    if (int rc = solo_batch(P)) return rc;
    Batch& B = *P->solo;
    bool changed = false;
    if (opts->local_solver == DDMGNN_LOCAL_LU) {
        if (int rc = prepare_exact(B, changed)) return rc;
    } else if (int rc = prepare_dss(B, opts->precision, changed)) {
        return rc;
    }
    DevProb v = make_view(P);
    v.r = const_cast<double*>(r);  // read only
    v.z = z;
    v.st = nullptr;
    HIP_TRY(launch_set_view(B.hook.p, v, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    const IterArgs ia = iter_args(*opts, -1);
    const DevProb* tab = B.hook.p;
    double* outs[3] = {local_ms, coarse_ms, glue_ms};
    hipEvent_t e0 = nullptr, e1 = nullptr;
    HIP_TRY(hipEventCreate(&e0));
    HIP_TRY(hipEventCreate(&e1));
    int rc = DDMGNN_OK;
    for (int stage = 0; stage < 3 && rc == DDMGNN_OK; ++stage) {
        if (stage == 1 && !opts->coarse) {
            if (outs[1]) *outs[1] = 0.0;
            continue;
        }
        hipGraph_t g = nullptr;
        hipGraphExec_t ge = nullptr;
        hipError_t he = hipStreamBeginCapture(ctx->cap, hipStreamCaptureModeRelaxed);
        if (he == hipSuccess) {
            ctx->launch = ctx->cap;
            for (int i = 0; i < reps && rc == DDMGNN_OK && he == hipSuccess; ++i) {
                if (stage == 0)
                    rc = enqueue_dss(B, tab, opts->precision, 1, true, opts->local_solver);
                else if (stage == 1)
                    he = launch_coarse(tab, B.coarse_rows.p, B.n_coarse, ctx->cap, false);
                else
                    he = launch_prolong(tab, B.vec_blk.p, B.n_vec, ia, ctx->cap, false);
            }
            ctx->launch = ctx->stream;
            const hipError_t ee = hipStreamEndCapture(ctx->cap, &g);
            if (he == hipSuccess) he = ee;
        }
        if (he == hipSuccess && rc == DDMGNN_OK) he = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
        if (g) (void)hipGraphDestroy(g);
        float ms = 0.f;
        if (he == hipSuccess && rc == DDMGNN_OK) {
            he = hipGraphLaunch(ge, ctx->stream);  // warm-up
            if (he == hipSuccess) he = hipEventRecord(e0, ctx->stream);
            if (he == hipSuccess) he = hipGraphLaunch(ge, ctx->stream);
            if (he == hipSuccess) he = hipEventRecord(e1, ctx->stream);
            if (he == hipSuccess) he = hipEventSynchronize(e1);
            if (he == hipSuccess) he = hipEventElapsedTime(&ms, e0, e1);
        }
        if (ge) (void)hipGraphExecDestroy(ge);
        if (he != hipSuccess && rc == DDMGNN_OK) rc = fail(DDMGNN_E_HIP, hipGetErrorString(he));
        if (rc == DDMGNN_OK && outs[stage]) *outs[stage] = (double)ms / reps;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return rc;
}

int ddmgnn_precond_apply(ddmgnn_ctx* ctx, ddmgnn_problem* P, const ddmgnn_solve_opts* opts, const double* r,
                         double* z) {
    if (!ctx || !P || !opts || !r || !z) return fail(DDMGNN_E_INVALID, "null argument");
    if (r == z) return fail(DDMGNN_E_INVALID, "r and z must not alias");
    if (int rc = check_opts(*opts)) return rc;
    if (int rc = solo_batch(P)) return rc;
    Batch& B = *P->solo;
    bool changed = false;
    if (opts->local_solver == DDMGNN_LOCAL_LU) {
        if (int rc = prepare_exact(B, changed)) return rc;
    } else if (int rc = prepare_dss(B, opts->precision, changed)) {
        return rc;
    }
    DevProb v = make_view(P);
    v.r = const_cast<double*>(r);  // read only: the apply never writes its input
    v.z = z;
    v.st = nullptr;
    HIP_TRY(launch_set_view(B.hook.p, v, ctx->stream));
    if (int rc = enqueue_apply(B, B.hook.p, *opts, -1, nullptr, false)) return rc;
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    return DDMGNN_OK;
}

int ddmgnn_apply_intermediates(ddmgnn_ctx* ctx, ddmgnn_problem* P, double* s, double* y0, double* y,
                               double* local) {
    if (!ctx || !P) return fail(DDMGNN_E_INVALID, "null argument");
    hipStream_t st = ctx->stream;
    const int K = P->hs.K;
    if (s) HIP_TRY(hipMemcpyAsync(s, P->s.p, K * sizeof(double), hipMemcpyDeviceToDevice, st));
    if (y0) HIP_TRY(hipMemcpyAsync(y0, P->y0.p, K * sizeof(double), hipMemcpyDeviceToDevice, st));
    if (y) HIP_TRY(hipMemcpyAsync(y, P->y.p, K * sizeof(double), hipMemcpyDeviceToDevice, st));
    if (local) HIP_TRY(hipMemcpyAsync(local, P->local.p, P->hs.sk * sizeof(double), hipMemcpyDeviceToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    return DDMGNN_OK;
}

int ddmgnn_solve(ddmgnn_ctx* ctx, ddmgnn_problem* P, const ddmgnn_solve_opts* opts, double* u_out,
                 ddmgnn_stats* stats) {
    if (!ctx || !P || !opts || !u_out) return fail(DDMGNN_E_INVALID, "null argument");
    if (int rc = check_opts(*opts)) return rc;
    if (int rc = solo_batch(P)) return rc;
    double* outs[1] = {u_out};
    return solve_batch(ctx, *P->solo, *opts, outs, stats);
}

int ddmgnn_solve_batch(ddmgnn_ctx* ctx, ddmgnn_problem* const* probs, int32_t n, const ddmgnn_solve_opts* opts,
                       double* const* u_out, ddmgnn_stats* stats) {
    if (!ctx || !probs || n < 1 || !opts || !u_out) return fail(DDMGNN_E_INVALID, "null argument or n < 1");
    if (int rc = check_opts(*opts)) return rc;
    for (int i = 0; i < n; ++i) {
        if (!probs[i] || !u_out[i]) return fail(DDMGNN_E_INVALID, "null problem or output");
        if (probs[i]->ctx != ctx) return fail(DDMGNN_E_INVALID, "problem belongs to another context");
        if (probs[i]->model->id != probs[0]->model->id)
            return fail(DDMGNN_E_INVALID, "all problems of a batch must share the model");
        for (int j = 0; j < i; ++j)
            if (probs[j] == probs[i]) return fail(DDMGNN_E_INVALID, "a problem appears twice in the batch");
    }
    if (n == 1) return ddmgnn_solve(ctx, probs[0], opts, u_out[0], stats);
    bool hit = ctx->last_batch && (int)ctx->last_batch->ids.size() == n;
    for (int i = 0; hit && i < n; ++i) hit = ctx->last_batch->ids[i] == probs[i]->id;
    if (!hit) {
        ctx->last_batch.reset();
        if (int rc = build_batch(ctx, probs, n, ctx->last_batch)) return rc;
    }
    return solve_batch(ctx, *ctx->last_batch, *opts, u_out, stats);
}

int ddmgnn_expand_overlap(int64_t n_nodes, int64_t n_tri, const int32_t* tri, const int32_t* part, int32_t n_part,
                          int32_t delta, int64_t** sub_ptr_out, int32_t** sub_nodes_out) {
    if (n_nodes <= 0 || n_tri <= 0 || !tri || !part || n_part <= 0 || delta < 0 || !sub_ptr_out || !sub_nodes_out)
        return fail(DDMGNN_E_INVALID, "invalid argument");
    for (int64_t t = 0; t < 3 * n_tri; ++t)
        if (tri[t] < 0 || tri[t] >= n_nodes) return fail(DDMGNN_E_INVALID, "triangle node id out of range");
    for (int64_t i = 0; i < n_nodes; ++i)
        if (part[i] < 0 || part[i] >= n_part) return fail(DDMGNN_E_INVALID, "part id out of range");
    std::vector<int64_t> sp;
    std::vector<int32_t> sn;
    expand_overlap(n_nodes, n_tri, tri, part, n_part, delta, sp, sn);
    auto* a = (int64_t*)std::malloc(sp.size() * sizeof(int64_t));
    auto* b = (int32_t*)std::malloc(std::max<size_t>(1, sn.size()) * sizeof(int32_t));
    if (!a || !b) {
        std::free(a);
        std::free(b);
        return fail(DDMGNN_E_NOMEM, "host allocation failed");
    }
    std::memcpy(a, sp.data(), sp.size() * sizeof(int64_t));
    std::memcpy(b, sn.data(), sn.size() * sizeof(int32_t));
    *sub_ptr_out = a;
    *sub_nodes_out = b;
    return DDMGNN_OK;
}

int ddmgnn_pou_weights(int64_t n_nodes, const uint8_t* dirichlet, int32_t n_sub, const int64_t* sub_ptr,
                       const int32_t* sub_nodes, double* weights_out) {
    if (n_nodes <= 0 || !dirichlet || n_sub <= 0 || !sub_ptr || !sub_nodes || !weights_out)
        return fail(DDMGNN_E_INVALID, "invalid argument");
    std::vector<int32_t> mult(n_nodes, 0);
    for (int64_t k = 0; k < sub_ptr[n_sub]; ++k) {
        if (sub_nodes[k] < 0 || sub_nodes[k] >= n_nodes) return fail(DDMGNN_E_INVALID, "node id out of range");
        mult[sub_nodes[k]]++;
    }
    for (int64_t k = 0; k < sub_ptr[n_sub]; ++k) {
        const int32_t v = sub_nodes[k];
        weights_out[k] = dirichlet[v] ? 0.0 : 1.0 / (double)mult[v];
    }
    return DDMGNN_OK;
}

int ddmgnn_expand_overlap_device(ddmgnn_ctx* ctx, int64_t n_nodes, int64_t n_tri, const int32_t* tri,
                                 const int32_t* part, const uint8_t* dirichlet, int32_t n_part, int32_t delta,
                                 int64_t* sub_ptr_out, int32_t* sub_nodes_out, double* weights_out, int64_t cap) {
    if (!ctx || n_nodes <= 0 || n_nodes > INT32_MAX || n_tri <= 0 || n_tri > INT32_MAX / 3 || !tri || !part ||
        !dirichlet || n_part <= 0 || delta < 0 || !sub_ptr_out || cap < 0 || (cap > 0 && (!sub_nodes_out || !weights_out)))
        return fail(DDMGNN_E_INVALID, "invalid argument");
    hipStream_t s = ctx->stream;
    const int64_t n = n_nodes;
    DevBuf<int> status;
    DevBuf<int32_t> tri_cnt, tri_list, sets0, sets1, part_cnt;
    DevBuf<int64_t> tri_ptr, sub_ptr;
    DevBuf<uint8_t> sz0, sz1;
    HIP_TRY(status.alloc(1));
    HIP_TRY(hipMemsetAsync(status.p, 0, sizeof(int), s));
    HIP_TRY(ov_check(tri, n_tri, part, n, n_part, status.p, s));
    int bad = 0;
    HIP_TRY(hipMemcpyAsync(&bad, status.p, sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (bad & 1) return fail(DDMGNN_E_INVALID, "triangle node id out of range");
    if (bad & 2) return fail(DDMGNN_E_INVALID, "part id out of range");
    HIP_TRY(tri_cnt.alloc((size_t)n));
    HIP_TRY(tri_ptr.alloc((size_t)n + 1));
    HIP_TRY(tri_list.alloc((size_t)(3 * n_tri)));
    HIP_TRY(sets0.alloc((size_t)n * OV_CAP));
    HIP_TRY(sets1.alloc((size_t)n * OV_CAP));
    HIP_TRY(sz0.alloc((size_t)n));
    HIP_TRY(sz1.alloc((size_t)n));
    HIP_TRY(part_cnt.alloc((size_t)n_part));
    HIP_TRY(sub_ptr.alloc((size_t)n_part + 1));
    HIP_TRY(hipMemsetAsync(tri_cnt.p, 0, (size_t)n * sizeof(int32_t), s));
    int32_t* sets = nullptr;
    uint8_t* sz = nullptr;
    HIP_TRY(ov_grow(tri, n_tri, part, n, delta, tri_cnt.p, tri_ptr.p, tri_list.p, sets0.p, sets1.p, sz0.p, sz1.p,
                    &sets, &sz, status.p, s));
    HIP_TRY(hipMemsetAsync(part_cnt.p, 0, (size_t)n_part * sizeof(int32_t), s));
    HIP_TRY(ov_count(sets, sz, n, n_part, part_cnt.p, sub_ptr.p, s));
    HIP_TRY(hipMemcpyAsync(sub_ptr_out, sub_ptr.p, ((size_t)n_part + 1) * sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipMemcpyAsync(&bad, status.p, sizeof(int), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (bad & 4) return fail(DDMGNN_E_INVALID, "a node belongs to more than 16 overlapping sub-meshes");
    int64_t kmax = 0;
    for (int32_t i = 0; i < n_part; ++i) kmax = std::max(kmax, sub_ptr_out[i + 1] - sub_ptr_out[i]);
    if (kmax > OV_SORT_MAX) return fail(DDMGNN_E_INVALID, "sub-mesh larger than the supported maximum (16384 nodes)");
    const int64_t sk = sub_ptr_out[n_part];
    if (sk > cap)
        return fail(DDMGNN_E_INVALID, "capacity below sub_ptr_out[n_part] (the number of sub-mesh slots); "
                                      "call again with cap >= sub_ptr_out[n_part]");
    HIP_TRY(hipMemsetAsync(part_cnt.p, 0, (size_t)n_part * sizeof(int32_t), s));
    HIP_TRY(ov_fill(sets, sz, n, dirichlet, n_part, sub_ptr.p, sk, part_cnt.p, sub_nodes_out, weights_out, s));
    HIP_TRY(hipStreamSynchronize(s));
    return DDMGNN_OK;
}

void ddmgnn_free(void* p) { std::free(p); }

}  // extern "C"

int ddmgnn_train_rhs(ddmgnn_ctx* ctx, ddmgnn_problem* P, const double* u, float* c_out) {
    if (!ctx || !P || !u || !c_out) return fail(DDMGNN_E_INVALID, "null argument");
    hipStream_t s = ctx->stream;
    if (P->tr_r.n < (size_t)P->hs.n) HIP_TRY(P->tr_r.alloc((size_t)P->hs.n));
    HIP_TRY(launch_train_rhs(P->rowptr.p, P->col.p, P->val.p, P->b.p, u, P->tr_r.p, (int)P->hs.n, P->sub_ptr.p,
                             P->sub_nodes.p, P->hs.K, c_out, s));
    HIP_TRY(hipStreamSynchronize(s));
    return DDMGNN_OK;
}

int ddmgnn_train_grad(ddmgnn_ctx* ctx, ddmgnn_problem* P, const ddmgnn_model_desc* md, const float* theta,
                      const int32_t* subs, int32_t n, const float* c, const int64_t* c_off, double scale,
                      float* grad, double* loss_out, double* gnorm_out) {
    if (!ctx || !P || !md || !theta || !subs || !c || !c_off || !grad) return fail(DDMGNN_E_INVALID, "null argument");
    if (md->d != D) return fail(DDMGNN_E_INVALID, "training supports the latent width d = 10 only");
    if (md->kbar < 1 || md->kbar > 64) return fail(DDMGNN_E_INVALID, "kbar must be in 1..64");
    if (n < 1) return fail(DDMGNN_E_INVALID, "at least one sample required");
    if (!(scale >= 0.0) || !std::isfinite(scale)) return fail(DDMGNN_E_INVALID, "scale must be finite and >= 0");
    for (int32_t i = 0; i < n; ++i) {
        if (subs[i] < 0 || subs[i] >= P->hs.K) return fail(DDMGNN_E_INVALID, "sub-mesh index out of range");
        if (P->hs.sub_ptr[subs[i] + 1] - P->hs.sub_ptr[subs[i]] > kMaxSubNodes)
            return fail(DDMGNN_E_INVALID, "training samples are limited to sub-meshes of at most 2048 nodes");
        if (c_off[i] < 0) return fail(DDMGNN_E_INVALID, "negative right-hand side offset");
    }
    if (int rc = prepare_train(P)) return rc;
    const int kb = md->kbar, ks = (kb + 3) / 4 * 4;
    hipStream_t s = ctx->stream;
    auto grow = [&](auto& buf, size_t n) {
        if (buf.n >= n) return hipSuccess;
        P->device_bytes -= buf.n * sizeof(*buf.p);
        const hipError_t e = buf.alloc(n);
        P->device_bytes += buf.n * sizeof(*buf.p);
        return e;
    };
    // Tiles of all samples; chunks of whole samples share the scratch region.
    std::vector<int4> items;
    std::vector<int32_t> chunk;  // first tile of each chunk, and the end
    // scratch, in floats: blobs, inputs, states, sender rows, sums, r, rho, gr, receiver rows, own values, accumulators
    constexpr int NP = 12;
    size_t off[NP + 1] = {0};
    for (int64_t cap = TRAIN_TILES;; cap /= 2) {
        items.clear();
        chunk.assign(1, 0);
        int64_t most = 0;
        for (int32_t i = 0; i < n; ++i) {
            const int32_t t0 = P->vt_first[subs[i]], t1 = t0 + sub_tiles(P, subs[i]);
            int64_t first = (int64_t)items.size() / 2;
            if (first + (t1 - t0) >= INT32_MAX / 2) return fail(DDMGNN_E_INVALID, "too many samples");
            if (first > chunk.back() && first - chunk.back() + (t1 - t0) > cap) chunk.push_back((int32_t)first);
            first -= chunk.back();  // within the chunk
            for (int32_t t = t0; t < t1; ++t) {
                const VtTile f = P->vt_tiles[t];
                const int2 o = P->tr_out_rows[t];
                items.push_back(make_int4(t, (int)(first - t0) * VT_TILE, f.z, f.w));
                items.push_back(make_int4(o.x, o.y, (int)(uint32_t)(uint64_t)c_off[i],
                                          (int)(uint32_t)((uint64_t)c_off[i] >> 32)));
            }
            most = std::max(most, first + (t1 - t0));
        }
        chunk.push_back((int32_t)(items.size() / 2));
        const size_t T = (size_t)most, lanes = T * VT_TILE;
        const size_t parts[NP] = {(size_t)kb * TRAIN_BLOB, 2 * lanes, (size_t)(kb + 1) * T * 256,
                                  (size_t)kb * (lanes + 1) * 2 * D, (size_t)kb * T * 320, lanes * ks, lanes * ks,
                                  lanes * ks, (lanes + 1) * 4 * D, (lanes + 1) * 4 * D, T * 1024,
                                  (size_t)(kb + 1) * train_workgroups(most) * TRAIN_ACC * 64};
        for (int i = 0; i < NP; ++i) off[i + 1] = off[i] + (parts[i] + 63) / 64 * 64;
        const hipError_t e = grow(P->tr_scratch, off[NP]);
        if (e == hipSuccess) break;
        if (e != hipErrorOutOfMemory || chunk.size() > (size_t)n) HIP_TRY(e);  // not one sample fits
    }
    const size_t n_red = (size_t)(kb + 1) * TRAIN_ACC * 64;
    size_t n_sse = 0;
    for (size_t q = 0; q + 1 < chunk.size(); ++q) n_sse += (size_t)train_sse_count(chunk[q + 1] - chunk[q], ks);
    HIP_TRY(grow(P->tr_items, items.size()));
    HIP_TRY(grow(P->tr_red, n_red));
    HIP_TRY(grow(P->tr_sse, n_sse));
    HIP_TRY(grow(P->tr_out, 2));
    HIP_TRY(upload_async(P->tr_items.p, items.data(), items.size() * sizeof(int4), s));
    float* f = P->tr_scratch.p;
    TrainArgs a{};
    a.kbar = kb;
    a.ks = ks;
    a.alpha = (float)md->alpha;
    a.info = P->vt_info;
    a.node = P->vt_node;
    a.pos = P->vt_pos;
    a.rin = P->tr_rin.p;
    a.rout = P->tr_rout.p;
    a.lm_ptr = P->lm_ptr.p;
    a.lm_col = P->lm_col.p;
    a.lm_val = P->lm_val.p;
    a.c = c;
    a.blobs = a.blobs_out = f;
    a.in = reinterpret_cast<float2*>(f + off[1]);
    a.h = f + off[2];
    a.q = f + off[3];
    a.m = f + off[4];
    a.r = f + off[5];
    a.rho = f + off[6];
    a.gr = f + off[7];
    a.pg[0] = f + off[8];
    a.pg[1] = f + off[9];
    a.own = f + off[10];
    a.part = f + off[11];
    a.sse = P->tr_sse.p;
    for (size_t q = 0; q + 1 < chunk.size(); ++q) {
        a.items = P->tr_items.p + 2 * (size_t)chunk[q];
        a.n_tiles = chunk[q + 1] - chunk[q];
        HIP_TRY(launch_train_grad(a, theta, P->tr_map.p, P->tr_red.p, q > 0, s));
        a.sse += train_sse_count(a.n_tiles, ks);
    }
    HIP_TRY(launch_train_reduce(P->tr_red.p, P->tr_ent.p, kb, scale, grad, P->tr_out.p, P->tr_sse.p, (int)n_sse, s));
    double out2[2];
    HIP_TRY(hipMemcpyAsync(out2, P->tr_out.p, sizeof(out2), hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    if (loss_out) *loss_out = scale * out2[1];
    if (gnorm_out) *gnorm_out = std::sqrt(out2[0]);
    if (!std::isfinite(out2[0]) || !std::isfinite(out2[1]))
        return fail(DDMGNN_E_NONFINITE, "training loss or gradient is not finite");
    return DDMGNN_OK;
}

int ddmgnn_adam_step(ddmgnn_ctx* ctx, float* theta, const float* grad, float* m, float* v, int64_t n, double gnorm,
                     int32_t t, double lr, double beta1, double beta2, double eps, double clip) {
    if (!ctx || !theta || !grad || !m || !v) return fail(DDMGNN_E_INVALID, "null argument");
    if (n < 1 || t < 1) return fail(DDMGNN_E_INVALID, "n >= 1 and step t >= 1 required");
    if (!(beta1 >= 0.0 && beta1 < 1.0 && beta2 >= 0.0 && beta2 < 1.0 && eps > 0.0 && lr >= 0.0))
        return fail(DDMGNN_E_INVALID, "0 <= beta < 1, eps > 0 and lr >= 0 required");
    if (!std::isfinite(gnorm) || gnorm < 0.0) return fail(DDMGNN_E_NONFINITE, "gradient norm is not finite");
    const double gs = clip > 0.0 && gnorm > clip ? clip / gnorm : 1.0;
    const double bc1 = 1.0 - std::pow(beta1, t), bc2 = 1.0 - std::pow(beta2, t);
    HIP_TRY(launch_adam(theta, grad, m, v, n, (float)gs, (float)lr, (float)beta1, (float)beta2, (float)bc1,
                        (float)bc2, (float)eps, ctx->stream));
    HIP_TRY(hipStreamSynchronize(ctx->stream));
    return DDMGNN_OK;
}
