"""Batched single steps on tiles (FP64 batches, small FP32 batches: up to three steps per
launch, 32 x 16 nodes of which 28 x 12 are stored): members below, at and around a tile's
outputs, every kind of end.

* the same bits for any grouping into calls, with and without graphs;
* the state of each member against the lone solver: both exchange every step's values as
  stored, so they differ by a few roundings a step at most (bound: 4 n u D after n steps, D the
  largest deviation from the rest state, as against the oracle);
* the gradient, its recomputed states from the same kernel, against the oracle's reverse pass
  (FP64 1e-10 of the largest value, FP32 relative L2 1e-4: the bounds of the adjoint tests).
"""
import numpy as np
import pytest

import oracle
from parity_util import Spec, rel_l2, say
from paper_1406_6438_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

W9 = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1406_6438_amd import lbm
    lbm.load()


SIZES = [(2, 1), (5, 3), (28, 12), (29, 13), (56, 25), (97, 64), (250, 131)]
ENDS = {"periodic": {}, "walls": dict(walls_x=True, walls_y=True, u_wall=(0.01, -0.02)),
        "open": dict(open_x=True, rho_in=1.01, u_in=0.03, rho_out=0.99, u_out=0.02),
        "inout_walls": dict(inout=True, walls_y=True, u_in=0.03, rho_out=0.99)}


@pytest.mark.parametrize("ends", sorted(ENDS))
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_batched_tile_steps(storage, ends):
    from paper_1406_6438_amd import lbm
    specs = [Spec(Lx=Lx, Ly=Ly, tau=0.6 + 0.05 * k, d_p=9.0, G=(2e-5, -1e-5), u0=(0.02, -0.01),
                  storage=storage, **ENDS[ends]) for k, (Lx, Ly) in enumerate(SIZES)]
    eps = [s.input_eps(0.4 + 0.55 * (0.5 + 0.5 * W.noise((s.Ly, s.Lx), 21 + s.Lx)))
           for s in specs]
    n = 53
    states = []
    for calls, graph in (([n], 24), ([1] * n, 0), ([2, 25, 4, 22], 4)):
        solvers = [lbm.Solver(s.gpu(), e) for s, e in zip(specs, eps)]
        b = lbm.Batch(solvers)
        b.configure(2 if storage == "f64" else 4, graph_steps=graph)
        for k in calls:
            b.step(k)
        states.append([s.get_state().cpu().numpy() for s in solvers])
        if not graph:
            J, g = b.grad(11, 5)
        b.close()
        for s in solvers:
            s.close()
    u = 2.0 ** -53 if storage == "f64" else 2.0 ** -24
    for k, (spec, e) in enumerate(zip(specs, eps)):
        assert all(np.array_equal(states[0][k], st[k]) for st in states[1:])
        s = lbm.Solver(spec.gpu(), e)
        s.step(n)
        f = s.get_state().cpu().numpy()
        s.close()
        D = max(np.abs(f - W9[:, None, None] * spec.rho0 * e).max(), 1e-3)
        err = np.abs(states[0][k] - f).max()
        Jo, go = oracle.grad_outlet_flux(spec.oracle(), e, 11)
        gk = g[k].double().cpu().numpy()
        eg = np.abs(gk - go).max() / np.abs(go).max() if storage == "f64" else rel_l2(gk, go)
        say(f"[batch tile {storage} {ends} {spec.Lx}x{spec.Ly}] state {err:.2e} (bound "
            f"{4 * n * u * D:.2e}), gradient {eg:.2e}")
        assert err <= 4 * n * u * D
        assert eg <= (1e-10 if storage == "f64" else 1e-4)
