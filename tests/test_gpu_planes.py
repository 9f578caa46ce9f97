"""Rows of one to several runs beside symmetry planes, against the oracle.

A run's record says whether its faces have PMC ghost images (smoother) and
which lanes may (residual and products); both differ from run to run only
where a row has more than one.  Part of an ellipsoid with planes at the low
sides, rows along x of one run, of several, and ending a lane into the next,
and rows along y and z between planes; element by element:

  * apply, residual and smoother on both levels, FP64 1e-12 and FP32 2e-5;
  * the two-level V-cycle, single and of three vectors, whose residual walks
    the runs, FP64 1e-12 and FP32 5e-5;
  * block solves with FP64 and FP32 Krylov bases, whose products walk the
    runs (FP32 input in the second case), by the residual of the oracle's
    rows: rtol 1e-9, the recomputed residual within twice that.
(The tolerances are those of test_gpu_parity.py and test_gpu_pmc.py.)
"""
import numpy as np
import pytest

from oracle import geometry as geo, symmetry as sym
import layout as lay

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIGMA = 2.0
CASES = [((16, 6, 4), (0, 1)), ((18, 6, 4), (0, 1)), ((34, 4, 6), (0, 1, 2)), ((50, 6, 4), (1, 2)), ((6, 34, 4), (0, 1, 2)),
         ((4, 6, 36), (0, 1))]


def rel_inf(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("nh,axes", CASES)
def test_rows_beside_planes(nh, axes):
    from paper_1301_3794_amd import dm
    print("[case] rows beside planes", nh, axes, flush=True)
    h = 1.0 / max(nh)
    nf = tuple(n * (2 if a in axes else 1) for a, n in enumerate(nh))
    fr_full = geo.fractions(geo.Ellipsoid([0.5 * n * h for n in nf], [0.46 * n * h if n > 12 else 0.8 * n * h for n in nf]),
                            nf, h)
    vc = sym.HalfVCycle(fr_full, nh, h, SIGMA, axes, 2)
    fr7 = lay.fractions_to_padded(vc.exts[0].half_fractions(fr_full), nh)
    geom = dm.user_fractions(fr7, bc_lo=tuple(dm.BC_PMC if a in axes else dm.BC_PEC for a in range(3)))

    def dev(v, n, dt):
        return torch.tensor(lay.faces_to_padded(v, n), dtype=dt, device="cuda")

    def back(v, n):
        return lay.faces_from_padded(v.double().cpu().numpy(), n)

    def rnd(L, seed):
        v = np.zeros(L.op.grid.n_faces)
        v[L.op.act] = np.random.default_rng(seed).standard_normal(L.op.act.size)
        return v

    with dm.Operator(geom, nh, h, SIGMA, levels=2) as op:
        n = nh
        for lev, L in enumerate(vc.levels):
            assert op.layout(lev)["active_faces"] == L.op.act.size
            x, f = rnd(L, 1), rnd(L, 2)
            for dt, tol in ((torch.float64, 1e-12), (torch.float32, 2e-5)):
                y = op.apply(dm.APPLY_M, dev(x, n, dt), op.face_tensor(level=lev, dtype=dt), level=lev)
                assert rel_inf(back(y, n)[L.op.act], (L.M @ x)[L.op.act]) <= tol
                r = op.residual(dev(f, n, dt), dev(x, n, dt), op.face_tensor(level=lev, dtype=dt), level=lev)
                assert rel_inf(back(r, n)[L.op.act], (f - L.M @ x)[L.op.act]) <= tol
                for reverse in (False, True):
                    xs = op.smooth(dev(f, n, dt), dev(x, n, dt), reverse=reverse, level=lev)
                    ref = x.copy()
                    vc._smooth(L, ref, f, vc.ORDER[::-1] if reverse else vc.ORDER)
                    assert rel_inf(back(xs, n), ref) <= tol
            n = tuple(v // 2 for v in n)
        L = vc.levels[0]
        fs = [rnd(L, 10 + q) for q in range(3)]
        for dt, tol in ((torch.float64, 1e-12), (torch.float32, 5e-5)):
            fd = [dev(f, nh, dt) for f in fs]
            xs = [op.vcycle(fd[0], op.face_tensor(dtype=dt))]
            xs += op.vcycle_block(fd, [op.face_tensor(dtype=dt) for _ in fd])
            for f, x in zip([fs[0]] + fs, xs):
                assert rel_inf(back(x, nh), vc(f)) <= tol
        for basis32, mode in ((0, dm.SOLVE_FGMRES_MG64), (0, dm.SOLVE_FGMRES_MG32), (1, dm.SOLVE_FGMRES_MG32)):
            with dm.Operator(geom, nh, h, SIGMA, levels=2, krylov_basis_f32=basis32) as sop:
                xs = [sop.face_tensor() for _ in fs]
                infos = sop.solve_block([dev(f, nh, torch.float64) for f in fs], xs, mode=mode, rtol=1e-9)
                w = np.sqrt(vc.exts[0].mult)   # the norm of the library: half of a face in a plane is owned
                for f, x, info in zip(fs, xs, infos):
                    assert info["status"] == 0
                    res = (f - L.M @ back(x, nh)) * w
                    assert np.linalg.norm(res[L.op.act]) <= 2e-9 * np.linalg.norm((f * w)[L.op.act])
