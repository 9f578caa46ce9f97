"""The row runs of the stencil kernels (16 lanes each) at row ends: rows
shorter than a run, of one, of several and ending a lane or two into the
next, and odd rows (the coarser level), against the oracle.

Tolerances (norm-wise, as in test_gpu_parity.py): FP64 1e-12, FP32 2e-5.
"""
import numpy as np
import pytest

from oracle import geometry as geo, multigrid as omg
import layout as lay

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rel_inf(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


def vec(level, seed):
    x = np.zeros(level.op.grid.n_faces)
    x[level.op.act] = np.random.default_rng(seed).standard_normal(level.op.act.size)
    return x


@pytest.mark.parametrize("nx", [6, 14, 18, 34, 66, 130])
def test_rows_of_every_run_width(nx):
    from paper_1301_3794_amd import dm
    n, h, sigma = (nx, 6, 4), 1.0 / nx, 2.0
    # wider than the box across x, so the rows hold vacuum stretches and cut ends
    fr = geo.fractions(geo.Ellipsoid((0.5, 3 * h, 2 * h), (0.46, 5 * h, 4 * h)), n, h)
    vc = omg.VCycle(fr, n, h, sigma, 2)
    with dm.Operator(dm.user_fractions(lay.fractions_to_padded(fr, n)), n, h, sigma, levels=2) as op:
        for lev, L in enumerate(vc.levels):
            print(f"[case] nx={nx} level={lev} n={L.n}", flush=True)
            x, f = vec(L, 1), vec(L, 2)
            for dt, tol in ((torch.float64, 1e-12), (torch.float32, 2e-5)):
                xd = torch.tensor(lay.faces_to_padded(x, L.n), dtype=dt, device="cuda")
                fd = torch.tensor(lay.faces_to_padded(f, L.n), dtype=dt, device="cuda")
                y = op.apply(dm.APPLY_M, xd, torch.full_like(xd, 7.0), level=lev)
                assert rel_inf(lay.faces_from_padded(y.double().cpu().numpy(), L.n)[L.op.act], (L.M @ x)[L.op.act]) <= tol
                r = op.residual(fd, xd, op.face_tensor(level=lev, dtype=dt), level=lev)
                assert rel_inf(lay.faces_from_padded(r.double().cpu().numpy(), L.n), f - L.M @ x) <= tol
                for reverse in (False, True):
                    xs = op.smooth(fd, xd.clone(), reverse=reverse, level=lev)
                    ref = x.copy()
                    vc._smooth(L, ref, f, vc.ORDER[::-1] if reverse else vc.ORDER)
                    assert rel_inf(lay.faces_from_padded(xs.double().cpu().numpy(), L.n), ref) <= tol
