"""Calls that the automatic choice of kernels must not make slower than the explicit ones it
chooses between (all of them give the same bits or results within rounding).

Each comparison times both sides in turn on the same lattice, best of several, and allows 20%:
the routes it tells apart differ by 40% and more (FP64 2048^2, one step: one-step sweep 104 us,
one-step tile 151; a tuned FP32 batch of 0.15M nodes: 5.3 us a step on sweeps, 2.5 on tiles);
6% where a step with its record is timed too (4096^2 FP32: 475 / 521).
"""
import dataclasses

import pytest

from parity_util import Spec, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1406_6438_amd import lbm
    lbm.load()


def _eps(Lx, Ly, storage, seed=1):
    g = torch.Generator(device="cuda").manual_seed(seed)
    e = 0.35 + 0.65 * torch.rand((Ly, Lx), device="cuda", generator=g, dtype=torch.float64)
    return e if storage == "f64" else e.float()


def _time(f, reps):
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(reps):
        f()
    b.record()
    torch.cuda.synchronize()
    return a.elapsed_time(b) * 1e3 / reps


def _compare(what, f, ref, reps, rounds=7, limit=1.2):
    """Best time of a call of f and of ref, taken in turn."""
    f(), ref()
    t = [(_time(f, reps), _time(ref, reps)) for _ in range(rounds)]
    tf, tr = min(x for x, _ in t), min(y for _, y in t)
    say(f"[routes] {what}: {tf:.2f} us, reference {tr:.2f} us")
    assert tf <= limit * tr, what


def _spec(L, storage, **kw):
    return Spec(Lx=L[0], Ly=L[1], tau=0.8, d_p=20.0, u0=(0.02, 0.0), walls_y=True,
                storage=storage, **kw)


@pytest.mark.parametrize("L, storage, every", [((2048, 2048), "f64", 0), ((512, 512), "f64", 0),
                                               ((4096, 4096), "f32", 2),
                                               ((1024, 1024), "f32", 2)])
def test_single_steps_are_not_slower_than_the_sweep(L, storage, every):
    """One step per call (or between two records) against the one-step sweep: on both sides
    of the size up to which a single step goes on tiles."""
    from paper_1406_6438_amd import lbm
    spec, eps = _spec(L, storage, diag_every=every), _eps(*L, storage)
    auto = lbm.Solver(spec.gpu(), eps)
    sweep = lbm.Solver(dataclasses.replace(spec, steps_per_pass=1).gpu(), eps)
    for s in (auto, sweep):
        s.step(2)
    per = max(every, 1)
    _compare(f"{storage} {L} every {every}", lambda: auto.step(per), lambda: sweep.step(per), 20,
             limit=1.06 if every and L[0] > 2048 else 1.2)
    # past the size the two kernels take turns: still the same bits
    auto.step(7)
    sweep.step(7)
    assert torch.equal(auto.get_state(), sweep.get_state())
    auto.close()
    sweep.close()


def test_batched_single_steps_are_not_slower_than_the_sweep():
    from paper_1406_6438_amd import lbm
    spec = _spec((1450, 725), "f64")
    for n in (1, 4):
        sv = [[lbm.Solver(spec.gpu(), _eps(1450, 725, "f64", k)) for k in range(n)]
              for _ in range(2)]
        auto, sweep = lbm.Batch(sv[0]), lbm.Batch(sv[1])
        sweep.configure(2, 0, 24, 1)
        _compare(f"batch of {n} f64", lambda: auto.step(1), lambda: sweep.step(1), 20)
        auto.step(7)
        sweep.step(7)
        for a, b in zip(*sv):
            assert torch.equal(a.get_state(), b.get_state())
        auto.close()
        sweep.close()
        for s in sv[0] + sv[1]:
            s.close()


def _members(storage, sizes):
    from paper_1406_6438_amd import lbm
    return [lbm.Solver(Spec(Lx=Lx, Ly=Lx // 2, tau=0.8, d_p=20.0, u0=(0.02, 0.0), walls_y=True,
                            inout=True, u_in=0.02, storage=storage).gpu(),
                       _eps(Lx, Lx // 2, storage, Lx)) for Lx in sizes]


@pytest.mark.parametrize("storage, sizes", [("f32", (129, 250, 470)), ("f32", (900, 1010)),
                                            ("f64", (129, 250, 470)), ("f64", (900, 1010)),
                                            ("f64", (9, 12)), ("f32", (2048, 2048, 1500))])
def test_tuned_batch_is_not_slower_than_an_untuned_one(storage, sizes):
    """The tuner's pick against the automatic configuration: steps (several graphs of them)
    and the gradient, whose recomputed states do not depend on the pick; and a batch
    configured with what the tuner returned runs what the tuner timed."""
    from paper_1406_6438_amd import lbm
    sv = [_members(storage, sizes) for _ in range(3)]
    tuned, auto, copied = (lbm.Batch(s) for s in sv)
    for b in (tuned, auto, copied):
        b.step(1)
    best, trials = tuned.tune(reps=10)
    assert best["us_per_step"] == min(t["us_per_step"] for t in trials)
    copied.configure(best["vec"], best["grid"], best["graph_steps"], best["steps_per_pass"],
                     best["pass_rows"])
    say(f"[routes] tuned {storage} {sizes}: {best}")
    _compare(f"tuned {storage} {sizes}", lambda: tuned.step(96), lambda: auto.step(96), 2)
    _compare(f"configured as tuned {storage} {sizes}", lambda: copied.step(96),
             lambda: tuned.step(96), 2)
    _compare(f"gradient of the tuned {storage} {sizes}", lambda: tuned.grad(60, 20),
             lambda: auto.grad(60, 20), 1, rounds=5)
    for b in (tuned, auto, copied):
        b.close()
    for s in sum(sv, []):
        s.close()
