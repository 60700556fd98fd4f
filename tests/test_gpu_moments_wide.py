"""The macroscopic fields on both sides of the size from which the read-out takes vectors of
nodes (a tile of 64 lanes x 4 rows for each of the 256 compute units; below, one node per
lane): ragged rows, walls, against the oracle's moments of the state the GPU gives out.

Bounds as for small lattices: 64 roundings in any field, 64 N in a sum over N nodes.
"""
import numpy as np
import pytest

import oracle
from parity_util import Spec, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1406_6438_amd import lbm
    lbm.load()


@pytest.mark.parametrize("ends", [{}, dict(walls_x=True, walls_y=True)], ids=["periodic", "walls"])
@pytest.mark.parametrize("storage, sizes", [("f64", [(128, 1020), (128, 1021), (515, 1030)]),
                                            ("f32", [(256, 1020), (254, 1021), (1021, 1030)]),
                                            ("f16", [(256, 1020), (253, 1021), (1023, 1030)])])
def test_moments_of_vectors(storage, sizes, ends):
    from paper_1406_6438_amd import lbm, workloads as W
    u = 2.0 ** -53 if storage == "f64" else 2.0 ** -24
    for Lx, Ly in sizes:
        spec = Spec(Lx=Lx, Ly=Ly, tau=0.7, d_p=9.0, G=(2e-5, -1e-5), u0=(0.02, -0.01),
                    storage=storage, **ends)
        eps = spec.input_eps(0.35 + 0.65 * (0.5 + 0.5 * W.noise((Ly, Lx), 77 + Lx)))
        s = lbm.Solver(spec.gpu(), eps)
        s.step(3)
        ref = oracle.moments(spec.oracle(), eps,
                             s.get_state().double().cpu().numpy().reshape(9, Ly, Lx))
        for diag in (True, False):
            m = s.moments(want_diag=diag)
            for name in ("eps_rho", "rho", "ux", "uy"):
                err = np.abs(m[name].double().cpu().numpy() - ref[name]).max()
                say(f"[moments {storage} {Lx}x{Ly}] {name} {err:.2e} (bound {64 * u:.2e})")
                assert err <= 64 * u
            if diag:
                rec, N = m["diag"], Lx * Ly
                assert abs(rec[0] - ref["eps_rho"].sum()) <= 64 * N * u
                assert abs(rec[3] - (ref["eps_rho"] * ref["ux"]).sum()) <= 64 * N * u
                assert abs(rec[5] - np.hypot(ref["ux"], ref["uy"]).max()) <= 64 * u
                assert rec[6] == 0 and rec[7] == 3
        s.close()
