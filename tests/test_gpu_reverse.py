"""The gradient's reverse steps on tiles (16 x 16 nodes, the inner 12 x 12 owned, up to three
steps per launch): lattices below, at and around a tile's outputs, every kind of end, against
the oracle's reverse pass (FP64 storage: 1e-10 of the largest value, FP32: relative L2 1e-4,
the bounds of the adjoint tests); and both sides of the largest plane the tiles address, past
which each launch takes one step on rows.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from parity_util import Spec, rel_l2, say
from paper_1406_6438_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1406_6438_amd import lbm
    lbm.load()


SIZES = [(2, 1), (5, 3), (12, 12), (13, 25), (16, 16), (37, 30)]
ENDS = {"periodic": {}, "walls_y": dict(walls_y=True, u_wall=(0.01, -0.02)),
        "walls": dict(walls_x=True, walls_y=True),
        "open": dict(open_x=True, rho_in=1.01, u_in=0.03, rho_out=0.99, u_out=0.02),
        "inout_walls": dict(inout=True, walls_y=True, u_in=0.03, rho_out=0.99)}


@pytest.mark.parametrize("ends", sorted(ENDS))
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_reverse_tiles(storage, ends):
    from paper_1406_6438_amd import lbm
    for Lx, Ly in SIZES:
        spec = Spec(Lx=Lx, Ly=Ly, tau=0.7, d_p=9.0, G=(2e-5, -1e-5), u0=(0.02, -0.01),
                    storage=storage, **ENDS[ends])
        eps = spec.input_eps(0.4 + 0.55 * (0.5 + 0.5 * W.noise((Ly, Lx), 55 + Lx)))
        Jo, go = oracle.grad_outlet_flux(spec.oracle(), eps, 11)
        for ckpt in (5, 11):                   # launches of 3 + 2 (and 1) and 3 + 3 + 3 + 2
            s = lbm.Solver(spec.gpu(), eps)
            J, g = s.grad(11, ckpt)
            g = g.double().cpu().numpy()
            s.close()
            err = (np.abs(g - go).max() / np.abs(go).max() if storage == "f64" else
                   rel_l2(g, go))
            say(f"[reverse {storage} {ends} {Lx}x{Ly} ckpt {ckpt}] {err:.2e}")
            assert err <= (1e-10 if storage == "f64" else 1e-4)


def test_largest_plane_of_the_reverse_tiles():
    """A channel periodic in y, its porosity repeated every 512 rows: the gradient repeats as
    well (FP32 adjoints: within 1e-6).  1024 x 262144 nodes are the first past the tiles'
    2^31 bytes of an FP64 plane; the last rows below and past it are compared with a lone
    period, and a batch with the large one takes the rows too."""
    from paper_1406_6438_amd import lbm
    n, P = 4, 512
    spec = Spec(Lx=1024, Ly=P, tau=0.7, d_p=9.0, u0=(0.02, 0.0), storage="f32", inout=True,
                u_in=0.02, steps_per_pass=1)
    eps = torch.tensor(0.4 + 0.55 * (0.5 + 0.5 * W.noise((P, 1024), 5)), dtype=torch.float32,
                       device="cuda")
    s = lbm.Solver(spec.gpu(), eps)
    J0, g0 = s.grad(n, n)
    s.close()
    g0 = g0.double()
    for periods in (511, 512):
        say(f"[largest reverse plane] 1024x{P * periods}")
        big = dataclasses.replace(spec, Ly=P * periods)
        assert (1024 * big.Ly * 8 < 2 ** 31) == (periods == 511)
        s = lbm.Solver(big.gpu(), eps.repeat(periods, 1))
        out = [s.grad(n, n)]
        if periods == 512:
            s.close()
            s = lbm.Solver(big.gpu(), eps.repeat(periods, 1))
            t = lbm.Solver(spec.gpu(), eps)
            b = lbm.Batch([s, t])
            b.configure(4, steps_per_pass=1)
            Js, gs = b.grad(n, n)
            out.append((Js[0], gs[0]))
            assert rel_l2(gs[1].double().cpu(), g0.cpu()) <= 1e-6
            b.close()
            t.close()
        s.close()
        for J, g in out:
            assert abs(J - periods * J0) <= 1e-6 * abs(periods * J0)
            for k in (0, 1, periods // 2, periods - 2, periods - 1):
                d = g[k * P:(k + 1) * P].double() - g0
                assert float(d.norm() / g0.norm()) <= 1e-6
        del s, out, J, g
        torch.cuda.empty_cache()
