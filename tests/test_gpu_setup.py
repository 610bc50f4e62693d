"""Setup on the device against independent host computations.

* Overlap expansion and partition-of-unity weights (Sec. II.A, overlap of
  Sec. IV.A): bit-exact against the oracle's decomposition (oracle.decomp).
* Coarse level (Sec. III.A step 1): the device forms R_0 A R_0^T and inverts
  it by blocked Gauss-Jordan; the coarse solve y = A_0^{-1} y0 of an apply is
  compared with numpy's solve of the oracle's A_0, on problems whose K spans
  many pivot blocks and tiles of the inversion.
* DDM-LU local solvers (eq. (7)): the device assembles and inverts every
  R_i A R_i^T; the local terms of an apply are compared with numpy's solve of
  the oracle's local matrices.
The tolerances are those of an explicitly formed inverse of order m applied
to a vector against a direct solve: m * eps * kappa relative to the largest
entry.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2402_08296_amd as dg  # noqa: E402
import workload as W  # noqa: E402
from oracle import decomp as dc, schwarz as sw  # noqa: E402
from tests._cases import oracle_problem  # noqa: E402

pytestmark = pytest.mark.gpu

SMOOTHER = W.smoother_theta(omega=0.15, out_scale=1.7)


@pytest.fixture(scope="module")
def ctx():
    print("[gpu] creating context", flush=True)
    return dg.Context()


def _i32(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("seed,n,parts,delta", [(1, 2500, 5, 2), (2, 4000, 9, 1), (3, 3000, 4, 4), (4, 6000, 12, 0),
                                                (5, 100_000, 150, 2)])
def test_overlap_expansion_on_device_bitexact(ctx, seed, n, parts, delta):
    p = W.make_problem(seed, n, parts, 0.3)
    print(f"[gpu] device overlap N={p.n} parts={parts} delta={delta}", flush=True)
    sp, nodes, w = ctx.expand_overlap_device(p.n, _i32(p.mesh.tri), _i32(p.part),
                                             torch.from_numpy(p.mesh.dirichlet.astype(np.uint8)).cuda(), parts, delta)
    dec = dc.decompose(p.n, p.mesh.tri, p.mesh.dirichlet, p.part, parts, delta)
    assert np.array_equal(sp, dec.sub_ptr)
    assert np.array_equal(nodes.cpu().numpy(), dec.sub_nodes)
    assert np.array_equal(w.cpu().numpy(), dec.weights)


def test_overlap_expansion_refuses_bad_ids(ctx):
    p = W.make_problem(1, 2000, 4, 0.3)
    bad = p.part.copy()
    bad[7] = 4
    with pytest.raises(dg.DDMGNNError, match="part id"):
        ctx.expand_overlap_device(p.n, _i32(p.mesh.tri), _i32(bad),
                                  torch.from_numpy(p.mesh.dirichlet.astype(np.uint8)).cuda(), 4, 2)
    tri = p.mesh.tri.copy()
    tri[3, 1] = p.n
    with pytest.raises(dg.DDMGNNError, match="triangle"):
        ctx.expand_overlap_device(p.n, _i32(tri), _i32(p.part),
                                  torch.from_numpy(p.mesh.dirichlet.astype(np.uint8)).cuda(), 4, 2)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("seed,n,parts,delta", [(11, 20_000, 40, 2), (12, 120_000, 700, 2), (15, 6000, 240, 4)])
def test_coarse_level_formed_on_device(ctx, seed, n, parts, delta):
    """y = A_0^{-1} R_0 r of one apply against numpy's solve of the oracle's A_0 (K = 40 and
    700: one and eleven pivot blocks of 64, up to 121 tiles of 64 x 64 per step). The third
    problem (small parts, overlap 4) has rows of A_0 with more than 32 nonzero columns, which
    the assembly sums on one thread, beside rows summed by whole workgroups."""
    p = W.make_problem(seed, n, parts, 0.3)
    hp = oracle_problem(p, delta=delta)
    print(f"[gpu] device coarse level N={p.n} K={hp.K}", flush=True)
    prob = dg.Problem(ctx, hp, dg.Model(ctx, SMOOTHER))
    A = p.A.to_scipy()
    dec = dc.Decomposition(p.n, hp.sub_ptr, hp.sub_nodes, hp.weights)
    co = sw.Coarse(A, dec)
    if delta == 4:
        assert (np.count_nonzero(co.A0, axis=1) > 32).any() and (np.count_nonzero(co.A0, axis=1) <= 32).any()
    r = p.b - A @ p.u0
    z = torch.empty(p.n, dtype=torch.float64, device="cuda")
    prob.apply(torch.from_numpy(r).cuda(), z, dg.default_opts(precision="fp64"))
    _, y0, y, _ = [t.cpu().numpy() for t in prob.intermediates()]
    y0_ref = co.Z.T @ r
    y_ref = np.linalg.solve(co.A0, y0_ref)
    err = np.abs(y - y_ref).max() / np.abs(y_ref).max()
    cond = np.linalg.cond(co.A0)
    print(f"[gpu]   coarse solve relative error {err:.2e} (cond(A_0) {cond:.1e})", flush=True)
    assert np.abs(y0 - y0_ref).max() <= 1e-12 * np.abs(y0_ref).max()
    assert err <= hp.K * np.finfo(float).eps * cond  # an inverse of order K against a direct solve


@pytest.mark.timeout(300)
def test_singular_coarse_refused_on_device(ctx):
    """Two identical sub-meshes make R_0 A R_0^T singular: problem creation reports E_NOT_SPD."""
    p = W.make_problem(13, 1800, 4, 0.2)
    hp = oracle_problem(p)
    sp = np.concatenate([hp.sub_ptr, [hp.sub_ptr[-1] + hp.sub_ptr[1]]])
    sn = np.concatenate([hp.sub_nodes, hp.sub_nodes[:hp.sub_ptr[1]]])
    w = np.concatenate([hp.weights, hp.weights[:hp.sub_ptr[1]]])
    w[:hp.sub_ptr[1]] *= 0.5
    w[hp.sub_ptr[-1]:] *= 0.5
    hp2 = dg.HostProblem(hp.xy, hp.tri, hp.dirichlet, hp.rowptr, hp.col, hp.val, hp.b, hp.u0, sp, sn, w)
    with pytest.raises(dg.DDMGNNError) as ei:
        dg.Problem(ctx, hp2, dg.Model(ctx, SMOOTHER))
    assert ei.value.code == -4


@pytest.mark.timeout(300)
def test_local_inverses_formed_on_device(ctx):
    """Local terms of a DDM-LU apply (the device inverses times R_i r) against numpy's solve
    of each R_i A R_i^T (every seventh sub-mesh; sub-meshes of 219 to 6102 nodes, up to 96
    pivot blocks of 64 in one batch)."""
    p = W.make_problem(14, 60_000, 60, 0.5)
    hp = oracle_problem(p)
    ks = np.diff(hp.sub_ptr)
    print(f"[gpu] device local inverses K={hp.K} k in [{ks.min()}, {ks.max()}]", flush=True)
    prob = dg.Problem(ctx, hp, dg.Model(ctx, SMOOTHER))
    A = p.A.to_scipy().tocsr()
    r = p.b - A @ p.u0
    z = torch.empty(p.n, dtype=torch.float64, device="cuda")
    prob.apply(torch.from_numpy(r).cuda(), z, dg.default_opts(local_solver=dg.LOCAL_LU,
                                                              prolong=dg.PROLONG_UNWEIGHTED))
    loc = prob.intermediates()[3].cpu().numpy()
    worst = 0.0
    for i in range(0, hp.K, 7):
        idx = hp.sub_nodes[hp.sub_ptr[i]:hp.sub_ptr[i + 1]]
        Ai = A[idx][:, idx].toarray()
        ref = np.linalg.solve(Ai, r[idx])
        err = np.abs(loc[hp.sub_ptr[i]:hp.sub_ptr[i + 1]] - ref).max() / np.abs(ref).max()
        worst = max(worst, err / (idx.size * np.finfo(float).eps * np.linalg.cond(Ai)))
    print(f"[gpu]   worst local error in units of k eps kappa: {worst:.2e}", flush=True)
    assert worst <= 1.0


def _split(sizes):
    """A 9k-node problem whose sub-meshes are consecutive runs of its nodes (free nodes first)
    of the given sizes, and one of the rest: disjoint, so every R_i A R_i^T and A_0 is SPD."""
    p = W.make_problem(16, 9000, 4, 0.2)
    hp = oracle_problem(p)
    nodes = np.argsort(p.mesh.dirichlet, kind="stable")
    sp = np.concatenate([[0], np.cumsum(sizes), [p.n]])
    for a, b in zip(sp[:-1], sp[1:]):
        nodes[a:b].sort()
    w = np.where(p.mesh.dirichlet[nodes], 0.0, 1.0)
    return p, dg.HostProblem(hp.xy, hp.tri, hp.dirichlet, hp.rowptr, hp.col, hp.val, hp.b, hp.u0, sp, nodes, w)


@pytest.mark.timeout(300)
@pytest.mark.parametrize("sizes", [[1, 2, 63, 64, 65], [127, 128, 129, 193], [1983, 1984, 2048], [1, 2047, 2049], [2113, 2]])
def test_local_inverses_at_tile_edges(ctx, sizes):
    """Local terms of a DDM-LU apply at orders around the 64 x 64 tiles of the inverses, of one
    row of tiles or of several (an odd and an even number), and on both sides of 2048 (one
    vector per wavefront in LDS or one wavefront per workgroup)."""
    p, hp = _split(sizes)
    print(f"[gpu] local inverses of orders {sizes}", flush=True)
    prob = dg.Problem(ctx, hp, dg.Model(ctx, SMOOTHER))
    A = p.A.to_scipy().tocsr()
    r = p.b - A @ p.u0
    z = torch.empty(p.n, dtype=torch.float64, device="cuda")
    prob.apply(torch.from_numpy(r).cuda(), z, dg.default_opts(local_solver=dg.LOCAL_LU,
                                                              prolong=dg.PROLONG_UNWEIGHTED))
    loc = prob.intermediates()[3].cpu().numpy()
    for i, k in enumerate(sizes):
        idx = hp.sub_nodes[hp.sub_ptr[i]:hp.sub_ptr[i + 1]]
        Ai = A[idx][:, idx].toarray()
        ref = np.linalg.solve(Ai, r[idx])
        err = np.abs(loc[hp.sub_ptr[i]:hp.sub_ptr[i + 1]] - ref).max() / np.abs(ref).max()
        assert err <= k * np.finfo(float).eps * np.linalg.cond(Ai), k


@pytest.mark.timeout(300)
@pytest.mark.parametrize("K", [2, 63, 64, 65, 128, 129])
def test_coarse_inverse_at_tile_edges(ctx, K):
    """y = A_0^{-1} R_0 r at orders around the 64 x 64 tiles of the coarse inversion."""
    p, hp = _split([60] * (K - 1))
    print(f"[gpu] coarse inverse of order {hp.K}", flush=True)
    prob = dg.Problem(ctx, hp, dg.Model(ctx, SMOOTHER))
    A = p.A.to_scipy()
    co = sw.Coarse(A, dc.Decomposition(p.n, hp.sub_ptr, hp.sub_nodes, hp.weights))
    r = p.b - A @ p.u0
    z = torch.empty(p.n, dtype=torch.float64, device="cuda")
    prob.apply(torch.from_numpy(r).cuda(), z, dg.default_opts(precision="fp64"))
    y = prob.intermediates()[2].cpu().numpy()
    ref = np.linalg.solve(co.A0, co.Z.T @ r)
    assert np.abs(y - ref).max() <= K * np.finfo(float).eps * np.linalg.cond(co.A0) * np.abs(ref).max()


def _local_terms_match(ctx, n, seed, sizes, which):
    p = W.make_problem(seed, n, 4, 0.2)
    hp = oracle_problem(p)
    nodes = np.argsort(p.mesh.dirichlet, kind="stable")
    sp = np.concatenate([[0], np.cumsum(sizes), [p.n]]) if sum(sizes) < p.n else np.concatenate([[0], np.cumsum(sizes)])
    for a, b in zip(sp[:-1], sp[1:]):
        nodes[a:b].sort()
    w = np.where(p.mesh.dirichlet[nodes], 0.0, 1.0)
    hp = dg.HostProblem(hp.xy, hp.tri, hp.dirichlet, hp.rowptr, hp.col, hp.val, hp.b, hp.u0, sp, nodes, w)
    prob = dg.Problem(ctx, hp, dg.Model(ctx, SMOOTHER))
    before = prob.device_bytes()
    A = p.A.to_scipy().tocsr()
    r = p.b - A @ p.u0
    z = torch.empty(p.n, dtype=torch.float64, device="cuda")
    prob.apply(torch.from_numpy(r).cuda(), z, dg.default_opts(local_solver=dg.LOCAL_LU, prolong=dg.PROLONG_UNWEIGHTED))
    s, _, _, loc = [t.cpu().numpy() for t in prob.intermediates()]
    for i in which:
        idx = hp.sub_nodes[sp[i]:sp[i + 1]]
        Ai = A[idx][:, idx].toarray()
        ref = np.linalg.solve(Ai, r[idx])
        err = np.abs(loc[sp[i]:sp[i + 1]] - ref).max() / np.abs(ref).max()
        assert err <= idx.size * np.finfo(float).eps * np.linalg.cond(Ai), idx.size
        assert s[i] == pytest.approx(np.linalg.norm(r[idx]), rel=1e-13)
    # a square per sub-mesh is counted, whatever form it is held in
    k = np.diff(sp).astype(np.int64)
    assert prob.device_bytes() - before == int((8 * k * ((k + 1) // 2 * 2) + 8).sum())


@pytest.mark.timeout(300)
@pytest.mark.parametrize("sizes", [[1, 1, 3, 16, 61, 64], [66, 127, 128, 129, 131, 192, 193], [201, 255, 256, 257], [7, 2048, 64]])
def test_small_local_inverses(ctx, sizes):
    """Local terms of a DDM-LU apply where inverses are held as squares (up to 256 nodes: one
    tile inverted in LDS, or packed from tiles; one or two strips of 128 columns), beside
    sub-meshes held in tiles."""
    print(f"[gpu] small local inverses of orders {sizes}", flush=True)
    _local_terms_match(ctx, 9000, 16, sizes, range(len(sizes)))


@pytest.mark.timeout(300)
def test_many_small_local_inverses(ctx):
    """More squares than are packed from one buffer of tiles (2048 of 65 nodes)."""
    print("[gpu] 2060 local inverses of order 65", flush=True)
    _local_terms_match(ctx, 140_000, 17, [65] * 2060, [0, 1, 2046, 2047, 2048, 2049, 2059])
