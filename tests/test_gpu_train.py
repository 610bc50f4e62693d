"""Training of DSS_theta on the GPU against the oracle: loss and gradient of the residual
loss summed over the blocks, the Adam step and the local right-hand sides."""
import numpy as np
import pytest

import paper_2402_08296_amd as dg
import workload as W
from oracle import decomp as dc
from oracle import dss
from oracle import train as tr
from tests._cases import small_problem

pytestmark = pytest.mark.gpu

# FP32 forward and backward over kbar blocks against FP64. Measured: loss 7e-8
# relative, gradient 3e-7 of its largest entry (kbar = 4, alpha = 0.3); the
# bounds keep a factor of about 70.
LOSS_RTOL = 2e-6
GRAD_ATOL = 2e-5


@pytest.fixture(scope="module")
def setup():
    import torch
    p, hp = small_problem()
    ctx = dg.Context()
    th0 = W.xavier_theta(0, 30, 10)
    model = dg.Model(ctx, th0)
    prob = dg.Problem(ctx, hp, model)
    A = p.A.to_scipy()
    subs = []
    for i in range(hp.K):
        nodes = hp.sub_nodes[hp.sub_ptr[i]:hp.sub_ptr[i + 1]]
        g = dc.local_graph(nodes, p.mesh.tri, p.mesh.xy, p.mesh.dirichlet)
        subs.append((nodes, g, tr.local_matrix(A, nodes)))
    yield p, hp, ctx, prob, subs, torch
    prob.close()
    model.close()
    ctx.close()


def _theta(seed, kbar, bias=0.3):
    rng = np.random.default_rng(seed)
    th = W.xavier_theta(seed, kbar, 10).astype(np.float64)
    th = th + bias * rng.standard_normal(th.size) * (th == 0)
    return th.astype(np.float32)


def _rhs(g, seed):
    c = np.random.default_rng(seed).standard_normal(g.k)
    c[g.dirichlet == 1] = 0.0
    return (c / np.linalg.norm(c)).astype(np.float32)


def _run(setup, kbar, alpha, theta, order, seeds):
    p, hp, ctx, prob, subs, torch = setup
    cs = [_rhs(subs[i][1], s) for i, s in zip(order, seeds)]
    offs = np.cumsum([0] + [c.size for c in cs[:-1]])
    cdev = torch.tensor(np.concatenate(cs), device="cuda")
    tdev = torch.tensor(theta, device="cuda")
    grad = torch.empty_like(tdev)
    loss, gn = prob.train_grad(tdev, order, cdev, offs, grad, kbar=kbar, alpha=alpha)
    scale = 1.0 / sum(c.size for c in cs)
    samples = [(subs[i][1], subs[i][2], c.astype(np.float64)) for i, c in zip(order, cs)]
    L, G = tr.loss_and_grad(theta.astype(np.float64), samples, alpha, kbar, 10, scale)
    return loss, gn, grad.cpu().numpy(), L, G


@pytest.mark.parametrize("kbar,alpha", [(4, 0.3), (30, 1e-3)])
def test_loss_and_gradient_match_oracle(setup, kbar, alpha):
    theta = _theta(1, kbar) if kbar < 30 else W.xavier_theta(3, 30, 10)
    order = [0, 2, 1, 3]
    loss, gn, g, L, G = _run(setup, kbar, alpha, theta, order, [11, 12, 13, 14])
    print(f"kbar={kbar}: loss rel err {abs(loss - L) / L:.2e}, grad err {np.abs(g - G).max() / np.abs(G).max():.2e}")
    assert abs(loss - L) <= LOSS_RTOL * L
    assert np.abs(g - G).max() <= GRAD_ATOL * np.abs(G).max()
    assert gn == pytest.approx(float(np.linalg.norm(g.astype(np.float64))), rel=1e-6)


def test_gradient_deterministic_and_sample_order(setup):
    """Two calls give the same bits; the sum over samples runs in sample order, and
    a batch equals the sum of its samples' gradients up to that order."""
    p, hp, ctx, prob, subs, torch = setup
    theta = _theta(2, 3)
    cs = [_rhs(subs[i][1], 20 + i) for i in range(2)]
    cdev = torch.tensor(np.concatenate(cs), device="cuda")
    tdev = torch.tensor(theta, device="cuda")
    offs = [0, cs[0].size]
    g1, g2 = torch.empty_like(tdev), torch.empty_like(tdev)
    l1, _ = prob.train_grad(tdev, [0, 1], cdev, offs, g1, kbar=3, alpha=0.3, scale=1.0)
    l2, _ = prob.train_grad(tdev, [0, 1], cdev, offs, g2, kbar=3, alpha=0.3, scale=1.0)
    assert l1 == l2 and torch.equal(g1, g2)
    ga, gb = torch.empty_like(tdev), torch.empty_like(tdev)
    la, _ = prob.train_grad(tdev, [0], cdev, [0], ga, kbar=3, alpha=0.3, scale=1.0)
    lb, _ = prob.train_grad(tdev, [1], cdev, [offs[1]], gb, kbar=3, alpha=0.3, scale=1.0)
    assert l1 == pytest.approx(la + lb, rel=1e-12)
    assert torch.allclose(g1, ga + gb, rtol=1e-5, atol=1e-6 * float(g1.abs().max()))


def test_zero_weights_closed_form(setup):
    """theta = 0: the loss is kbar * scale * |c|^2 and only the decoders' output biases
    see a gradient, -2 scale sum_j (A_i c)_j."""
    p, hp, ctx, prob, subs, torch = setup
    kbar = 5
    c = _rhs(subs[1][1], 7)
    tdev = torch.zeros(dss.n_weights(kbar, 10), dtype=torch.float32, device="cuda")
    grad = torch.empty_like(tdev)
    loss, _ = prob.train_grad(tdev, [1], torch.tensor(c, device="cuda"), [0], grad, kbar=kbar, scale=0.5)
    c64 = c.astype(np.float64)
    assert loss == pytest.approx(kbar * 0.5 * float(c64 @ c64), rel=1e-6)
    g = grad.cpu().numpy()
    per = dss.n_weights(1, 10)
    ends = [k * per + per - 1 for k in range(kbar)]
    expect = -2 * 0.5 * float((subs[1][2] @ c64).sum())
    assert np.allclose(g[ends], expect, rtol=1e-5)
    assert np.abs(np.delete(g, ends)).max() == 0.0


def test_adam_step_matches_oracle(setup):
    p, hp, ctx, prob, subs, torch = setup
    rng = np.random.default_rng(5)
    n = 3 * dss.n_weights(1, 10)
    th, g = rng.standard_normal(n).astype(np.float32), (1e-2 * rng.standard_normal(n)).astype(np.float32)
    m = (1e-3 * rng.standard_normal(n)).astype(np.float32)
    v = (1e-5 * rng.random(n)).astype(np.float32)
    T = {k: torch.tensor(a, device="cuda") for k, a in dict(th=th, g=g, m=m, v=v).items()}
    gn = float(np.linalg.norm(g.astype(np.float64)))
    dg.adam_step(ctx, T["th"], T["g"], T["m"], T["v"], gn, 7, lr=1e-2, clip=1e-2)
    eth, em, ev = tr.adam_step(th.astype(np.float64), g.astype(np.float64), m.astype(np.float64),
                               v.astype(np.float64), 7, 1e-2, clip=1e-2)
    assert np.allclose(T["m"].cpu().numpy(), em, rtol=1e-5, atol=1e-9)
    assert np.allclose(T["v"].cpu().numpy(), ev, rtol=1e-5, atol=1e-12)
    assert np.abs(T["th"].cpu().numpy() - eth).max() <= 1e-5 * 1e-2 + 1e-6 * np.abs(eth).max()


def test_local_rhs_matches_oracle(setup):
    p, hp, ctx, prob, subs, torch = setup
    rng = np.random.default_rng(9)
    u = p.u0 + 0.1 * rng.standard_normal(p.n) * (p.mesh.dirichlet == 0)
    c = torch.empty(hp.sub_ptr[-1], dtype=torch.float32, device="cuda")
    prob.train_rhs(torch.tensor(u, device="cuda"), c)
    c = c.cpu().numpy()
    A = p.A.to_scipy()
    for i, (nodes, g, Ai) in enumerate(subs):
        e = tr.local_rhs(A, p.b, u, nodes)
        got = c[hp.sub_ptr[i]:hp.sub_ptr[i + 1]]
        assert np.abs(got - e).max() <= 1e-6 * np.abs(e).max()


def test_invalid_training_arguments(setup):
    p, hp, ctx, prob, subs, torch = setup
    tdev = torch.zeros(dss.n_weights(2, 10), dtype=torch.float32, device="cuda")
    grad = torch.empty_like(tdev)
    c = torch.zeros(4096, dtype=torch.float32, device="cuda")
    with pytest.raises((dg.DDMGNNError, ValueError)):
        prob.train_grad(tdev, [hp.K], c, [0], grad, kbar=2)
    with pytest.raises((dg.DDMGNNError, ValueError)):
        prob.train_grad(tdev, [0], c, [-1], grad, kbar=2)
    with pytest.raises((dg.DDMGNNError, ValueError)):
        prob.train_grad(torch.zeros(10 * 2 * 5, dtype=torch.float32, device="cuda"), [0], c, [0],
                        torch.zeros(100, dtype=torch.float32, device="cuda"), kbar=2, d=5)


def test_harvest_matches_oracle_pcg_iterates(setup):
    """Samples harvested at DDM-LU-PCG iterates equal the oracle's local right-hand sides
    at the oracle's PCG iterates (FP64 iterates agree to rounding)."""
    from oracle import krylov as kr, schwarz as sw
    from paper_2402_08296_amd import train as T
    p, hp, ctx, prob, subs, torch = setup
    its = [0, 1, 3]
    h = T.harvest(prob, its)
    A = p.A.to_scipy()
    dec = dc.Decomposition(p.n, hp.sub_ptr, hp.sub_nodes, hp.weights)
    M = sw.DDMLU(A, p.mesh.dirichlet, dec, prolong="unweighted")
    c = h.c.cpu().numpy()
    for t, it in enumerate(its):
        u = p.u0 if it == 0 else kr.pcg(A, p.b, p.u0, M, 1e-300, max_it=it).u
        for i, (nodes, g, Ai) in enumerate(subs):
            e = tr.local_rhs(A, p.b, u, nodes)
            got = c[t * h.sum_k + hp.sub_ptr[i]:t * h.sum_k + hp.sub_ptr[i + 1]]
            assert np.abs(got - e).max() <= 1e-5 * np.abs(e).max(), (it, i)
    assert len(h.samples()) == len(its) * hp.K


def test_training_lowers_the_loss(setup):
    """A few epochs of Adam (lr 1e-2, clipping 1e-2, batches of 4) from Xavier weights lower
    the epoch loss, and theta stays finite."""
    from paper_2402_08296_amd import train as T
    p, hp, ctx, prob, subs, torch = setup
    h = T.harvest(prob, [0, 2])
    st = T.init_state(torch.tensor(W.xavier_theta(8, 5, 10), device="cuda"))
    losses = [T.train_epoch(ctx, [(prob, h)], st, batch=4, kbar=5, alpha=0.3, seed=e) for e in range(6)]
    print("epoch losses", ["%.4g" % x for x in losses])
    assert losses[-1] < 0.9 * losses[0]
    assert bool(torch.isfinite(st.theta).all())
    assert st.step == 6 * ((len(h.samples()) + 3) // 4)


def test_many_samples_run_in_chunks(setup):
    """600 samples run as launches of 512 sharing one scratch region: the loss and gradient
    equal those of the two parts computed separately (up to the order of the sample sum)."""
    p, hp, ctx, prob, subs, torch = setup
    cs = [_rhs(subs[i][1], 40 + i) for i in range(hp.K)]
    starts = np.cumsum([0] + [c.size for c in cs[:-1]])
    cdev = torch.tensor(np.concatenate(cs), device="cuda")
    theta = torch.tensor(_theta(6, 2), device="cuda")
    order = [i % hp.K for i in range(600)]
    offs = [int(starts[i]) for i in order]
    g, ga, gb = (torch.empty_like(theta) for _ in range(3))
    L, _ = prob.train_grad(theta, order, cdev, offs, g, kbar=2, alpha=0.3, scale=1e-3)
    La, _ = prob.train_grad(theta, order[:512], cdev, offs[:512], ga, kbar=2, alpha=0.3, scale=1e-3)
    Lb, _ = prob.train_grad(theta, order[512:], cdev, offs[512:], gb, kbar=2, alpha=0.3, scale=1e-3)
    assert L == pytest.approx(La + Lb, rel=1e-12)
    assert torch.allclose(g, ga + gb, rtol=1e-5, atol=1e-6 * float(g.abs().max()))
    # repeated samples contribute identical terms: L = sum_i count_i L_i over the sub-meshes
    g1 = torch.empty_like(theta)
    per = [prob.train_grad(theta, [i], cdev, [int(starts[i])], g1, kbar=2, alpha=0.3, scale=1e-3)[0]
           for i in range(hp.K)]
    assert L == pytest.approx(sum(order.count(i) * per[i] for i in range(hp.K)), rel=1e-12)


def test_largest_sub_mesh_matches_oracle(setup):
    """A sub-mesh of exactly 2048 nodes (the library's limit) against the oracle."""
    p0, hp0, ctx, prob0, subs0, torch = setup
    p = W.make_problem(11, 5400, 3, 0.0)
    hp = dg.host_problem(p.mesh.xy, p.mesh.tri, p.mesh.dirichlet, p.A.rowptr, p.A.col, p.A.val, p.b, p.u0,
                         p.part, p.n_parts, 2)
    sizes = np.diff(hp.sub_ptr)
    big = int(np.argmax(sizes))
    assert sizes[big] == 2048
    model = dg.Model(ctx, W.xavier_theta(0, 30, 10))
    prob = dg.Problem(ctx, hp, model)
    nodes = hp.sub_nodes[hp.sub_ptr[big]:hp.sub_ptr[big + 1]]
    g = dc.local_graph(nodes, p.mesh.tri, p.mesh.xy, p.mesh.dirichlet)
    Ai = tr.local_matrix(p.A.to_scipy(), nodes)
    c = _rhs(g, 77)
    theta = _theta(9, 2)
    grad = torch.empty(theta.size, dtype=torch.float32, device="cuda")
    loss, _ = prob.train_grad(torch.tensor(theta, device="cuda"), [big], torch.tensor(c, device="cuda"), [0], grad,
                              kbar=2, alpha=0.3)
    L, G = tr.loss_and_grad(theta.astype(np.float64), [(g, Ai, c.astype(np.float64))], 0.3, 2, 10, 1.0 / g.k)
    gg = grad.cpu().numpy()
    print(f"k=2048: loss rel err {abs(loss - L) / L:.2e}, grad err {np.abs(gg - G).max() / np.abs(G).max():.2e}")
    assert abs(loss - L) <= LOSS_RTOL * L
    assert np.abs(gg - G).max() <= GRAD_ATOL * np.abs(G).max()
    prob.close()
    model.close()


def test_chunks_and_tile_edges_match_oracle_sums(setup):
    """More tiles than one scratch region holds: the batch is run in two chunks and equals the
    sum of its parts; a batch of one sample repeated gives the same gradient as that sample
    once (scale 1/n), whatever tiles of a workgroup the copies fall on."""
    p, hp, ctx, prob, subs, torch = setup
    theta = torch.tensor(_theta(5, 2), device="cuda")
    cs = [_rhs(subs[i][1], 40 + i) for i in range(hp.K)]
    cdev = torch.tensor(np.concatenate(cs), device="cuda")
    off = np.cumsum([0] + [c.size for c in cs[:-1]])
    tiles = [(c.size + 15) // 16 for c in cs]
    n = 32768 // min(tiles) + 3
    order = np.arange(n) % hp.K
    g, one = torch.empty_like(theta), torch.empty_like(theta)
    loss, _ = prob.train_grad(theta, order, cdev, off[order], g, kbar=2, alpha=0.3, scale=1e-3)
    assert sum(tiles[i] for i in order) > 32768
    want, total = torch.zeros_like(theta, dtype=torch.float64), 0.0
    for i in range(hp.K):
        L, _ = prob.train_grad(theta, [i], cdev, [off[i]], one, kbar=2, alpha=0.3, scale=1e-3)
        want += int((order == i).sum()) * one.double()
        total += int((order == i).sum()) * L
    assert loss == pytest.approx(total, rel=1e-6)
    # FP32 sums over the nodes in another order: the bar of the oracle comparison
    assert float((g.double() - want).abs().max()) <= GRAD_ATOL * float(want.abs().max())


def test_scratch_is_counted_and_kept(setup):
    """The scratch of a gradient call stays with the problem and shows in its device bytes: 4 bytes
    for about 1,000 kbar values per tile; a smaller call after it needs nothing more."""
    p, hp, ctx, prob, subs, torch = setup
    fresh = dg.Problem(ctx, hp, dg.Model(ctx, W.xavier_theta(0, 30, 10)))
    kbar = 4
    theta = torch.tensor(_theta(5, kbar), device="cuda")
    cs = [_rhs(subs[i][1], 60 + i) for i in range(hp.K)]
    cdev = torch.tensor(np.concatenate(cs), device="cuda")
    off = np.cumsum([0] + [c.size for c in cs[:-1]])
    order = np.arange(3 * hp.K) % hp.K
    g = torch.empty_like(theta)
    base = fresh.device_bytes()
    fresh.train_grad(theta, order, cdev, off[order], g, kbar=kbar, alpha=0.3)
    tiles = sum((cs[i].size + 15) // 16 for i in order)
    used = fresh.device_bytes() - base
    assert used >= 4 * 1000 * kbar * tiles
    fresh.train_grad(theta, [0], cdev, [off[0]], g, kbar=kbar, alpha=0.3)
    assert fresh.device_bytes() == base + used


def test_repeated_sample_gives_its_gradient(setup):
    """A batch of one sample repeated, with scale 1/n, gives that sample's gradient with scale 1,
    whatever tiles of a workgroup the copies fall on (one chunk and two)."""
    p, hp, ctx, prob, subs, torch = setup
    theta = torch.tensor(_theta(5, 2), device="cuda")
    c = _rhs(subs[1][1], 70)
    cdev = torch.tensor(c, device="cuda")
    tiles = (c.size + 15) // 16
    one, g = torch.empty_like(theta), torch.empty_like(theta)
    L, _ = prob.train_grad(theta, [1], cdev, [0], one, kbar=2, alpha=0.3, scale=1.0)
    for n in (2, 9, 32768 // tiles + 2):
        loss, _ = prob.train_grad(theta, np.full(n, 1), cdev, np.zeros(n, np.int64), g, kbar=2, alpha=0.3, scale=1.0 / n)
        assert loss == pytest.approx(L, rel=1e-6)  # the loss is scaled too
        # FP32 sums over the nodes in another order: the bar of the oracle comparison
        assert float((g - one).abs().max()) <= GRAD_ATOL * float(one.abs().max())
