"""Several single steps per launch on tiles (lbm_vans_step where a pass takes one step: FP64
storage, FP32 lattices too small for the multi-step passes, and the steps between recorded
states): 16 x 16 tiles with six steps per launch while every tile has a compute unit to
itself, else 32 x 16 tiles with five, four or three; FP32 lattices up to 2^20 nodes take
them with three steps.

Each size is run in one call, in calls of one step and in calls of uneven lengths: the
same bits, since a tile exchanges every step's values as they would have been stored.  The
state is held to the oracle by the bounds of one step per launch: FP64 a few ulp per step;
FP32 each step rounds each stored deviation once plus a few roundings in the collision,
4 n 2^-24 D after n steps (D the largest deviation from the rest state).
"""
import dataclasses

import numpy as np
import pytest

from parity_util import Spec, gpu_run, oracle_run, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

W9 = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1406_6438_amd import lbm
    lbm.load()


# sizes around the outputs of a tile (16 x 16, six steps: 6 x 6; 32 x 16: 24 x 8, 26 x 10,
# 28 x 12), below a tile, one column or row, and large enough for each tile shape
SIZES = {"f64": [(2, 1), (5, 3), (6, 6), (7, 13), (33, 17), (97, 64), (241, 131), (330, 205),
                 (521, 301)],
         "f32": [(2, 1), (13, 40), (97, 64), (250, 131), (523, 301)]}
ENDS = {"periodic": {}, "walls": dict(walls_x=True, walls_y=True, u_wall=(0.01, -0.02)),
        "open_walls": dict(open_x=True, walls_y=True, rho_in=1.01, u_in=0.03, rho_out=0.99,
                           u_out=0.02),
        "inout": dict(inout=True, u_in=0.03, rho_out=0.99)}


@pytest.mark.parametrize("ends", sorted(ENDS))
@pytest.mark.parametrize("storage, L", [(s, L) for s in SIZES for L in SIZES[s]])
def test_tile_steps(storage, L, ends):
    from paper_1406_6438_amd import lbm, workloads as W
    Lx, Ly = L
    spec = Spec(Lx=Lx, Ly=Ly, tau=0.7, d_p=9.0, G=(2e-5, -1e-5), u0=(0.02, -0.01),
                storage=storage, **ENDS[ends])
    eps = 0.35 + 0.65 * (0.5 + 0.5 * W.noise((Ly, Lx), 1234 + Lx))
    n = 17
    _, f = gpu_run(spec, eps, n)
    for calls in ([1] * n, [3, 7, 1, 6]):
        s = lbm.Solver(spec.gpu(), spec.input_eps(eps))
        for k in calls:
            s.step(k)
        g = s.get_state().cpu().numpy()
        s.close()
        assert np.array_equal(f, g)
    _, fo = oracle_run(spec, eps, n)
    e = spec.input_eps(eps)
    D = np.abs(fo - W9[:, None, None] * spec.rho0 * e).max()
    bound = 1e-13 if storage == "f64" else 4 * n * 2.0 ** -24 * max(D, 1e-3)
    say(f"[tile {storage} {Lx}x{Ly} {ends}] max |f - f_oracle| {np.abs(f - fo).max():.2e} "
        f"(bound {bound:.2e})")
    assert np.abs(f - fo).max() <= bound


@pytest.mark.parametrize("storage", ["f64", "f32"])
def test_records_between_tile_steps(storage):
    """Records of a run whose steps between the recorded states go several per launch, in
    calls that end off the records, against one-step launches: the same steps, and sums
    within the roundings of n steps over all nodes (9 values of size D rounded once a step
    and node, a few roundings each: 40 n N u D)."""
    from paper_1406_6438_amd import lbm, workloads as W
    Lx, Ly, n = 190, 77, 23
    spec = Spec(Lx=Lx, Ly=Ly, tau=0.7, d_p=9.0, G=(2e-5, 0.0), u0=(0.02, 0.0), storage=storage,
                walls_y=True, diag_every=5)
    eps = W.grf_porosity(Lx, Ly, seed=9, ell=4.0, lo=0.4, hi=1.0)
    out = []
    for per, calls in ((1, [n]), (0, [n]), (0, [4, 9, 1, 9])):
        s = lbm.Solver(dataclasses.replace(spec, steps_per_pass=per).gpu(), spec.input_eps(eps))
        for k in calls:
            s.step(k)
        rec, rc = s.diag_records()
        assert rc == 0
        out.append(rec)
        s.close()
    assert np.array_equal(out[1], out[2])
    assert np.array_equal(out[0][:, 7], [0, 5, 10, 15, 20]) and out[1].shape == out[0].shape
    u = 2.0 ** -53 if storage == "f64" else 2.0 ** -24
    bound = 40 * n * Lx * Ly * u * 0.05
    err = np.abs(out[1] - out[0]).max()
    say(f"[tile records {storage}] {err:.2e} (bound {bound:.2e})")
    assert err <= bound


def test_tile_gradient_is_the_same_for_any_checkpoints():
    """The gradient's forward and its recomputed states take the same tiles: the same bits
    for any checkpoint interval, and within 1e-10 of the gradient on one-step sweeps."""
    from paper_1406_6438_amd import lbm, workloads as W
    spec = Spec(Lx=61, Ly=34, tau=0.7, d_p=9.0, u0=(0.02, 0.0), storage="f64", walls_y=True,
                inout=True, u_in=0.02)
    eps = W.grf_porosity(61, 34, seed=5, ell=4.0, lo=0.4, hi=1.0)
    out = []
    for ckpt, per in ((29, 0), (7, 0), (1, 0), (7, 1)):
        s = lbm.Solver(dataclasses.replace(spec, steps_per_pass=per).gpu(), eps)
        out.append(s.grad(29, ckpt))
        s.close()
    for J, g in out[1:3]:
        assert J == out[0][0] and torch.equal(g, out[0][1])
    err = float((out[3][1] - out[0][1]).abs().max() / out[0][1].abs().max())
    say(f"[tile gradient] against one-step sweeps: {err:.2e}")
    assert err <= 1e-10
