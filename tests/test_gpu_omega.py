"""The multi-step passes and the batched tiles over the whole range of tau (below 1, above 1,
above 2) and under both drag laws.

* A shear mode of a uniform fluid at rest (eps = 1, no drag, no force; deviations +a along one
  diagonal, -a along the other) has no moments: each step multiplies it by 1 - omega and nothing
  else.  tau is chosen so that omega is an odd multiple of 2^-24 close to 1, where that last bit
  of FP32 omega is 64 2^-24 of 1 - omega: n steps must give (1 - omega)^n a to 4 n 2^-24 of it.
* States against the oracle within FP32 roundoff, 4 per step, of the largest stored magnitude
  (the bound of the parity tests).
"""
import dataclasses

import numpy as np
import pytest

import oracle
from parity_util import Spec, exec_mode, oracle_run, say
from paper_1406_6438_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

MODES = ["quads", "tall", "triples", "short", "tiny", "pairs", "wide", "auto"]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1406_6438_amd import lbm
    lbm.load()


@pytest.mark.parametrize("mode", MODES)
def test_shear_mode_decays_by_one_minus_omega(mode):
    from paper_1406_6438_amd import lbm
    omc, a, n = (2 ** 18 + 1) * 2.0 ** -24, 2.0 ** -7, 2 if mode == "pairs" else 4 if mode == "quads" else 3
    spec = Spec(Lx=96, Ly=40, tau=1.0 / (1.0 - omc), storage="f32", **exec_mode(mode, "f32"))
    eps = np.ones((40, 96))
    f = oracle.init(spec.oracle(), eps)
    d = np.array([0, 0, 0, 0, 0, a, -a, a, -a])[:, None, None]
    s = lbm.Solver(spec.gpu(), eps)
    s.set_state(f + d)
    s.step(n)
    # plain populations: the mode is what opposite diagonals hold more than the others
    g = s.get_state().cpu().numpy()
    s.close()
    want = omc ** n * a
    # get_state adds the rest state back in FP64: 2^-53 of 1/36 at most
    got = (g[5] + g[7] - g[6] - g[8]) / 4
    say(f"[shear mode {mode}] {np.abs(got / want - 1).max():.2e} (bound "
        f"{4 * n * 2.0 ** -24 + 2.0 ** -56 / want:.2e})")
    assert np.abs(got - want).max() <= 4 * n * 2.0 ** -24 * want + 2.0 ** -56


def _case(Lx, Ly, tau, drag, ends, storage="f32"):
    law = dict(drag_const=True, K=40.0, F_eps=0.4) if drag == "const" else dict(d_p=9.0)
    kw = {"periodic": dict(G=(2e-5, -1e-5)), "walls": dict(walls_x=True, walls_y=True,
                                                           G=(2e-5, -1e-5)),
          "inout_walls": dict(inout=True, walls_y=True, u_in=0.02, rho_out=0.995)}[ends]
    spec = Spec(Lx=Lx, Ly=Ly, tau=tau, u0=(0.02, 0.0), storage=storage, **law, **kw)
    return spec, spec.input_eps(W.grf_porosity(Lx, Ly, seed=31 + Lx, ell=4.0, lo=0.4, hi=1.0))


def _bound(spec, eps, fo, n):
    rest = oracle.init(dataclasses.replace(spec, u0=(0.0, 0.0)).oracle(), eps)
    de = max(np.abs(eps - np.roll(eps, s, axis=a)).max() for a in (0, 1) for s in (1, -1))
    return 4 * (n + 1) * 2.0 ** -24 * (np.abs(fo - rest).max() + de / 18.0)


@pytest.mark.parametrize("tau", [0.52, 1.3, 1.97, 2.6, 5.7])
@pytest.mark.parametrize("drag", ["ergun", "const"])
@pytest.mark.parametrize("ends", ["periodic", "walls", "inout_walls"])
def test_multi_step_passes_over_tau(ends, drag, tau):
    from paper_1406_6438_amd import lbm
    n = 13
    base, eps = _case(150, 61, tau, drag, ends)
    _, fo = oracle_run(base, eps, n)
    for mode in MODES:
        spec = dataclasses.replace(base, **exec_mode(mode, "f32"))
        s = lbm.Solver(spec.gpu(), eps)
        s.step(n)
        f = s.get_state().cpu().numpy()
        s.close()
        err, bound = np.abs(f - fo).max(), _bound(spec, eps, fo, n)
        say(f"[tau {tau} {drag} {ends} {mode}] {err:.2e} (bound {bound:.2e})")
        assert err <= bound, mode


@pytest.mark.parametrize("storage", ["f64", "f32"])
@pytest.mark.parametrize("ends", ["periodic", "walls", "inout_walls"])
def test_batched_constant_permeability(ends, storage):
    """Batched tiles, three- and four-step passes under the constant-K law."""
    from paper_1406_6438_amd import lbm
    n = 13
    cases = [_case(Lx, Ly, tau, "const", ends, storage)
             for Lx, Ly, tau in ((29, 40, 0.6), (97, 64, 1.4), (150, 41, 2.6))]
    ref = [oracle_run(spec, eps, n)[1] for spec, eps in cases]
    for per in ((0,) if storage == "f64" else (0, 2, 3, 4)):
        sv = [lbm.Solver(spec.gpu(), eps) for spec, eps in cases]
        b = lbm.Batch(sv)
        b.configure(2 if storage == "f64" else 4, 0, 0, per, 24 if per == 3 else 0)
        b.step(n)
        for (spec, eps), s, fo in zip(cases, sv, ref):
            err = np.abs(s.get_state().cpu().numpy() - fo).max()
            bound = 1e-13 if storage == "f64" else _bound(spec, eps, fo, n)
            say(f"[batch const K {storage} {ends} {per} {spec.Lx}x{spec.Ly}] {err:.2e} "
                f"(bound {bound:.2e})")
            assert err <= bound
        b.close()
        for s in sv:
            s.close()
