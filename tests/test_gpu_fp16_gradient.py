"""The gradient of FP16 runs (FP16 states decoded into the reverse tiles' FP64 arithmetic, FP32
adjoints between the launches), lone and batched, against 64-bit reverse steps on the CPU at the
very states the GPU stored: the FP16 rounding of the trajectory is then on both sides, and what
is left is one FP32 rounding per adjoint and step and a few FP64 ones.  Bound: 16 n 2^-24 of the
largest value after n steps.  The J of FP64 and FP32 runs on reverse tiles against the oracle's
(1e-12, 1e-5 of it: the adjoint tests' bounds).

Single steps, so that the states of the run and those the gradient recomputes are the same;
lattices below and above a reverse tile (12 x 12 owned of 16 x 16 nodes), with and without tiles
clear of every end.
"""
import pytest

import oracle
from parity_util import Spec, say
from paper_1406_6438_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1406_6438_amd import lbm
    lbm.load()


SIZES = [(5, 3), (13, 25), (61, 40)]
ENDS = {"periodic": {}, "walls": dict(walls_x=True, walls_y=True, u_wall=(0.01, -0.02)),
        "open_walls": dict(open_x=True, walls_y=True, u_in=0.02, u_out=0.02),
        "inout": dict(inout=True, u_in=0.03, rho_out=0.99)}
N = 11


def _case(ends, Lx, Ly, storage="f16", tau=0.7):
    spec = Spec(Lx=Lx, Ly=Ly, tau=tau, d_p=9.0, u0=(0.02, 0.0), storage=storage,
                G=(0.0, 0.0) if ends in ("open_walls", "inout") else (2e-5, -1e-5), **ENDS[ends])
    return spec, spec.input_eps(0.4 + 0.55 * (0.5 + 0.5 * W.noise((Ly, Lx), 55 + Lx)))


def _stored_states(solvers, stepper):
    """f(., 0 .. N) of each solver as the GPU holds them, one step per launch of the stepper
    (the lone sweep and the batched one are two compilations, which may fuse other
    multiply-adds, and a last bit moves whole FP16 roundings: each has states of its own)."""
    out = [[s.get_state().cpu() for s in solvers]]
    for _ in range(N):
        stepper.step(1)
        out.append([s.get_state().cpu() for s in solvers])
    return list(zip(*out))


def _reference(spec, eps, states):
    """dJ/deps by reverse steps of the 64-bit method at the given states."""
    from perf.cases import _Exact
    c = dict(bc_x="inout" if spec.inout else "open" if spec.open_x else
             "walls" if spec.walls_x else "periodic", bc_y="walls" if spec.walls_y else "periodic")
    p = spec.gpu()
    e = torch.tensor(eps, dtype=torch.float64, requires_grad=True)

    def back(out, ins, bar=None):
        return torch.autograd.grad(out, ins, bar, allow_unused=True)

    x, f = _Exact(c, p, e), states[-1].clone().requires_grad_(True)
    S, _, ux = x.moments(f)[:3]
    J = (S * ux)[:, -1].sum()
    lam, g = back(J, (f, e))
    for state in reversed(states[:-1]):
        x, f = _Exact(c, p, e), state.clone().requires_grad_(True)
        lam, ge = back(x.step(f), (f, e), lam)
        g = g + ge
    return g + back(_Exact(c, p, e).f, (e,), lam)[0]


def _check(what, g, go):
    err = float((g.double().cpu() - go).abs().max() / go.abs().max())
    say(f"[fp16 gradient {what}] {err:.2e} (bound {16 * N * 2.0 ** -24:.2e})")
    assert err <= 16 * N * 2.0 ** -24


@pytest.mark.parametrize("ends", sorted(ENDS))
def test_fp16_gradient(ends):
    from paper_1406_6438_amd import lbm
    cases = [_case(ends, Lx, Ly, tau=0.6 + 0.2 * k) for k, (Lx, Ly) in enumerate(SIZES)]
    for spec, eps in cases:
        s = lbm.Solver(spec.gpu(), eps)
        ref = _reference(spec, eps, _stored_states([s], s)[0])
        for ckpt in (5, N):
            _check(f"{ends} {spec.Lx}x{spec.Ly} ckpt {ckpt}", s.grad(N, ckpt)[1], ref)
        s.close()
    sv = [lbm.Solver(spec.gpu(), eps) for spec, eps in cases]
    b = lbm.Batch(sv)
    b.configure(4, 0, 0, 1)
    states = _stored_states(sv, b)
    for (spec, eps), g, st in zip(cases, b.grad(N, 4)[1], states):
        _check(f"{ends} {spec.Lx}x{spec.Ly} batch", g, _reference(spec, eps, st))
    b.close()
    for s in sv:
        s.close()


@pytest.mark.parametrize("ends", sorted(ENDS))
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_objective_of_the_reverse_tiles(storage, ends):
    from paper_1406_6438_amd import lbm
    for k, (Lx, Ly) in enumerate(SIZES):
        spec, eps = _case(ends, Lx, Ly, storage, 0.6 + 0.2 * k)
        Jo, _ = oracle.grad_outlet_flux(spec.oracle(), eps, N)
        s = lbm.Solver(spec.gpu(), eps)
        J, _ = s.grad(N, 5)
        b = lbm.Batch([s])
        Jb, _ = b.grad(N, 5)
        b.close()
        s.close()
        say(f"[objective {storage} {ends} {Lx}x{Ly}] {abs(J - Jo) / abs(Jo):.1e}, batch "
            f"{abs(Jb[0] - Jo) / abs(Jo):.1e}")
        for v in (J, Jb[0]):
            assert abs(v - Jo) <= (1e-12 if storage == "f64" else 1e-5) * abs(Jo)
