"""GPU: the scalar kernels of restarted FGMRES at the edges of their work split.

Sixteen wavefronts sum the Gram coefficients of a step, one each, and one
thread rotates the column and back-substitutes from LDS: cycles of one step, of
a whole round of wavefronts and one more or less, and the largest. A fixed
number of steps from the same start gives the oracle's iterate; the bar is
that of the solves to 1e-10 (1e-8 relative), which classical Gram-Schmidt run
twice and the oracle's modified one meet with eps times the basis' order to spare.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2402_08296_amd as dg  # noqa: E402
import workload as W  # noqa: E402
from oracle import decomp as dc, krylov as kr, schwarz as sw  # noqa: E402
from tests._cases import oracle_problem  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    print("[gpu] creating context", flush=True)
    p = W.make_problem(31, 4000, 6, 0.3)
    hp = oracle_problem(p)
    ctx = dg.Context()
    prob = dg.Problem(ctx, hp, dg.Model(ctx, W.smoother_theta(omega=0.15, out_scale=1.7)))
    dec = dc.Decomposition(p.n, hp.sub_ptr, hp.sub_nodes, hp.weights)
    return p, prob, sw.DDMLU(p.A.to_scipy(), p.mesh.dirichlet, dec, prolong="pou")


@pytest.mark.parametrize("restart,steps", [(1, 3), (2, 5), (15, 17), (16, 18), (17, 17), (33, 34), (64, 20), (64, 34)])
def test_fgmres_steps_match_oracle(setup, restart, steps):
    p, prob, M = setup
    print(f"[gpu] FGMRES({restart}), {steps} steps", flush=True)
    u, v = (torch.empty(p.n, dtype=torch.float64, device="cuda") for _ in range(2))
    o = dict(krylov=dg.FGMRES, restart=restart, local_solver=dg.LOCAL_LU, rtol=1e-14, max_it=steps)
    st = prob.solve(u, dg.default_opts(**o), check=False)
    prob.solve(v, dg.default_opts(graph=0, **o), check=False)
    ref = kr.fgmres(p.A.to_scipy(), p.b, p.u0, M, 1e-14, max_it=steps, restart=restart)
    assert st.iterations == ref.iterations == steps and torch.equal(u, v)
    assert np.linalg.norm(u.cpu().numpy() - ref.u) <= 1e-8 * np.linalg.norm(ref.u)
