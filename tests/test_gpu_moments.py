"""The macroscopic fields and diagnostics of a state, on the vector kernel: lattices of ragged
rows (the last lane of a run with fewer nodes, rows that start off a vector's boundary), one
row, one column, outputs off a vector's boundary and left out, every storage and end.

The reference is the oracle's moments of the state the GPU itself gives out.  Bounds: the sums
of nine values, the porosity gradient and the closed-form velocity are some 30 operations on
terms of size one at most, divided by a porosity of at least 0.35: below 64 roundings of size
2^-24 (FP32, and FP16, which computes in FP32) or 2^-53 (FP64) in any field.  The sums of the
diagnostics: those of each node, 64 N roundings.
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


SIZES = [(2, 1), (1, 7), (5, 3), (64, 9), (130, 4), (257, 33), (1020, 21)]
ENDS = {"periodic": {}, "walls": dict(walls_x=True, walls_y=True),
        "open_walls": dict(open_x=True, walls_y=True, rho_in=1.01, u_in=0.03, rho_out=0.99,
                           u_out=0.02),
        "inout": dict(inout=True, u_in=0.03, rho_out=0.99)}
FIELDS = ("eps_rho", "rho", "ux", "uy")


@pytest.mark.parametrize("ends", sorted(ENDS))
@pytest.mark.parametrize("storage", ["f64", "f32", "f16"])
def test_moments_of_ragged_rows(storage, ends):
    from paper_1406_6438_amd import lbm, workloads as W
    u = 2.0 ** -53 if storage == "f64" else 2.0 ** -24
    dt = torch.float64 if storage == "f64" else torch.float32
    for Lx, Ly in SIZES:
        if Lx == 1 and ends != "walls":
            continue
        spec = Spec(Lx=Lx, Ly=Ly, tau=0.7, d_p=9.0, G=(2e-5, -1e-5), u0=(0.02, -0.01),
                    storage=storage, **ENDS[ends])
        eps = spec.input_eps(0.35 + 0.65 * (0.5 + 0.5 * W.noise((Ly, Lx), 77 + Lx)))
        s = lbm.Solver(spec.gpu(), eps)
        s.step(3)
        ref = oracle.moments(spec.oracle(), eps,
                             s.get_state().double().cpu().numpy().reshape(9, Ly, Lx))
        got = []
        for off, diag in ((0, True), (1, True), (0, False)):
            flat = [torch.full((Lx * Ly + 2,), 7.0, dtype=dt, device="cuda") for _ in FIELDS]
            out = [f[off:off + Lx * Ly] for f in flat]
            rec, rc = lbm.lbm_vans_moments(s.h, *out, want_diag=diag)
            assert rc in (lbm.OK, lbm.WMACH)
            for f, o in zip(flat, out):        # nothing written around the field
                assert f[:off].eq(7.0).all() and f[off + Lx * Ly:].eq(7.0).all()
            got.append(([o.double().cpu().numpy().reshape(Ly, Lx) for o in out], rec))
        only = torch.empty(Lx * Ly, dtype=dt, device="cuda")
        lbm.lbm_vans_moments(s.h, None, None, only, None, want_diag=False)
        assert np.array_equal(only.double().cpu().numpy().reshape(Ly, Lx), got[2][0][2])
        s.close()
        for (f0, f1) in zip(got[0][0], got[1][0]):
            assert np.array_equal(f0, f1)
        assert np.array_equal(got[0][1], got[1][1])
        for fields, rec in got:
            for name, f in zip(FIELDS, fields):
                err = np.abs(f - ref[name]).max()
                say(f"[moments {storage} {ends} {Lx}x{Ly}] {name} {err:.2e} (bound {64 * u:.2e})")
                assert err <= 64 * u
        rec = got[0][1]
        er, ux, uy = ref["eps_rho"], ref["ux"], ref["uy"]
        N = Lx * Ly
        assert abs(rec[0] - er.sum()) <= 64 * N * u
        assert abs(rec[3] - (er * ux).sum()) <= 64 * N * u
        assert abs(rec[4] - (er * uy).sum()) <= 64 * N * u
        assert abs(rec[5] - np.sqrt(ux ** 2 + uy ** 2).max()) <= 64 * u
        assert rec[6] == 0 and rec[7] == 3
