"""A run of single steps (FP64, and FP32 lattices too small for the multi-step passes) is the
same to the bit whichever kernel takes a step: the one-step sweep of any width, the sweep that
also records diagnostics, or a tile of several steps.  So the state depends neither on how
often it is recorded, nor on how its steps are grouped into calls, nor on whether the lattice
runs alone or in a batch, and the gradient's forward ends in the same state.

Lattices below, at and around a tile's outputs, ragged rows, every kind of end, both drag
laws.  The comparison is of bits, so there is no tolerance.
"""
import dataclasses

import numpy as np
import pytest

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


SIZES = [(2, 1), (5, 3), (28, 12), (97, 64), (250, 131)]
ENDS = {"periodic": {}, "walls": dict(walls_x=True, walls_y=True, u_wall=(0.01, -0.02)),
        "open_walls": dict(open_x=True, walls_y=True, rho_in=1.01, u_in=0.03, rho_out=0.99,
                           u_out=0.02),
        "inout": dict(inout=True, u_in=0.03, rho_out=0.99)}
DRAG = {"ergun": dict(d_p=9.0), "const": dict(drag_const=True, K=40.0, F_eps=0.4)}
N = 13


def _case(storage, ends, drag, Lx, Ly, tau):
    spec = Spec(Lx=Lx, Ly=Ly, tau=tau, G=(2e-5, -1e-5), u0=(0.02, -0.01), storage=storage,
                **ENDS[ends], **DRAG[drag])
    return spec, spec.input_eps(0.35 + 0.65 * (0.5 + 0.5 * W.noise((Ly, Lx), 91 + Lx)))


def _state(spec, eps, calls=(N,)):
    from paper_1406_6438_amd import lbm
    s = lbm.Solver(spec.gpu(), eps)
    for k in calls:
        s.step(k)
    f = s.get_state()
    s.close()
    return f


@pytest.mark.parametrize("drag", sorted(DRAG))
@pytest.mark.parametrize("ends", sorted(ENDS))
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_state_is_the_same_for_any_kernel_of_single_steps(storage, ends, drag):
    vmax = 2 if storage == "f64" else 4
    for k, (Lx, Ly) in enumerate(SIZES):
        spec, eps = _case(storage, ends, drag, Lx, Ly, 0.56 + 0.3 * k)
        f = _state(spec, eps)
        assert torch.isfinite(f).all()
        kinds = {"sweeps": dict(steps_per_pass=1), "narrow": dict(steps_per_pass=1, sweep_vec=1),
                 "wide": dict(steps_per_pass=1, sweep_vec=vmax), "recorded": dict(diag_every=1),
                 "every 2": dict(diag_every=2), "every 5": dict(diag_every=5),
                 "recorded sweeps": dict(diag_every=3, steps_per_pass=1)}
        for name, kw in kinds.items():
            g = _state(dataclasses.replace(spec, **kw), eps)
            say(f"[single steps {storage} {ends} {drag} {Lx}x{Ly}] {name}: "
                f"same bits {torch.equal(f, g)}")
            assert torch.equal(f, g), name
        assert torch.equal(f, _state(dataclasses.replace(spec, diag_every=4), eps, [1] * N))


@pytest.mark.parametrize("ends", sorted(ENDS))
@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_batch_takes_the_lone_solvers_single_steps(storage, ends):
    from paper_1406_6438_amd import lbm
    cases = [_case(storage, ends, "ergun", Lx, Ly, 0.56 + 0.3 * k)
             for k, (Lx, Ly) in enumerate(SIZES)]
    ref = [_state(spec, eps) for spec, eps in cases]
    vmax = 2 if storage == "f64" else 4
    for cfg, calls in ((None, [N]), ((vmax, 0, 0), [1] * N), ((1, 0, 0, 1), [N]),
                       ((2, 8, 4, 1), [N]), ((vmax, 0, 4, 1), [N])):
        sv = [lbm.Solver(spec.gpu(), eps) for spec, eps in cases]
        b = lbm.Batch(sv)
        if cfg:
            b.configure(*cfg)
        for k in calls:
            b.step(k)
        same = [torch.equal(s.get_state(), r) for s, r in zip(sv, ref)]
        say(f"[single steps, batch {storage} {ends}] {cfg}: same bits {same}")
        b.close()
        for s in sv:
            s.close()
        assert all(same), cfg


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_gradient_forward_ends_in_the_state_of_the_steps(storage):
    """The gradient's last state is the one that the same steps give, and J the same value for
    any checkpoint interval, recorded or not, on sweeps and on tiles."""
    from paper_1406_6438_amd import lbm
    spec, eps = _case(storage, "inout", "ergun", 97, 64, 0.8)
    s = lbm.Solver(spec.gpu(), eps)
    s.step(N)
    f = s.get_state()
    s.close()
    out = []
    for ckpt, every, per in ((N, 0, 0), (4, 0, 0), (4, 3, 0), (4, 0, 1), (4, 2, 1)):
        s = lbm.Solver(dataclasses.replace(spec, diag_every=every, steps_per_pass=per).gpu(), eps)
        J, g = s.grad(N, ckpt)
        assert torch.equal(s.get_state(), f), (ckpt, every, per)
        s.close()
        out.append((J, g))
        assert J == out[0][0]
    assert torch.equal(out[2][1], out[1][1])   # the same launches, recorded or not


@pytest.mark.parametrize("storage, L", [("f16", (2048, 1024)), ("f32", (2048, 1024)),
                                        ("f32", (512, 300)), ("f64", (97, 64))])
def test_gradient_does_not_depend_on_recording(storage, L):
    """A gradient records nothing, so its passes (several steps each for the larger lattices)
    are those of a handle without diagnostics: the same bits of J, gradient and last state."""
    from paper_1406_6438_amd import lbm
    spec, eps = _case(storage, "inout", "ergun", *L, 0.8)
    out = []
    for every in (0, 5):
        s = lbm.Solver(dataclasses.replace(spec, diag_every=every).gpu(), eps)
        J, g = s.grad(12, 6)
        out.append((J, g, s.get_state()))
        s.close()
    say(f"[gradient {storage} {L}] J {out[0][0]!r} {out[1][0]!r}")
    assert out[0][0] == out[1][0]
    assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][2], out[1][2])


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_records_do_not_depend_on_the_launches(storage):
    """The recorded states are the same bits whatever takes the steps between them, and one
    kernel records them all: the same records, to the bit; the largest speed is the oracle's to
    64 roundings a step."""
    import oracle
    from paper_1406_6438_amd import lbm
    spec, eps = _case(storage, "walls", "ergun", 190, 77, 0.7)
    out = []
    for per, calls in ((1, [23]), (0, [23]), (0, [4, 9, 1, 9])):
        s = lbm.Solver(dataclasses.replace(spec, diag_every=5, steps_per_pass=per).gpu(), eps)
        for k in calls:
            s.step(k)
        rec, rc = s.diag_records()
        s.close()
        assert rc == 0 and np.array_equal(rec[:, 7], [0, 5, 10, 15, 20])
        out.append(rec)
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
    u = 2.0 ** -53 if storage == "f64" else 2.0 ** -24
    f = oracle.init(spec.oracle(), eps)
    for k, rec in enumerate(out[0]):
        m = oracle.moments(spec.oracle(), eps, f)
        top = np.hypot(m["ux"], m["uy"]).max()
        say(f"[records {storage}] n = {5 * k}: largest speed {rec[5]:.8f}, off by "
            f"{abs(rec[5] - top):.1e}")
        assert abs(rec[5] - top) <= 64 * (5 * k + 1) * u * 0.05 and rec[6] == 0
        f = oracle.steps(spec.oracle(), eps, f, 5)
