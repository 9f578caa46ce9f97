"""Block solves where the Gram-Schmidt passes change their form within a solve.

The passes of all systems share launches while a system has at most 32 columns
and the systems' bases together at most 128 MiB; beyond either the systems go
one by one.  A solve that crosses a limit has both forms on one case; a system
solved alone has only the second.  Iterations equal, solutions equal to 1e-12
(the sums are the same; a block's widest template may order them differently).
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,sigma,levels,nb,basis32,mode,rtol,crosses", [
    (16, 120.0, 2, 2, 0, "mg32", 1e-9, "columns"),
    (16, 120.0, 2, 3, 1, "mg32", 1e-9, "columns"),
    (64, 5.0, 0, 4, 0, "mg64", 1e-11, "bytes"),
])
def test_both_forms_in_one_solve(n, sigma, levels, nb, basis32, mode, rtol, crosses):
    from paper_1301_3794_amd import dm
    print("[case] block solve", n, nb, basis32, crosses, flush=True)
    m = {"mg32": dm.SOLVE_FGMRES_MG32, "mg64": dm.SOLVE_FGMRES_MG64}[mode]
    geom = dm.ellipsoid((0.5, 0.5, 0.5), (0.45, 0.41, 0.38))
    with dm.Operator(geom, (n,) * 3, 1.0 / n, sigma, levels=levels, nu_pre=1, nu_post=1, fgmres_restart=100,
                     krylov_basis_f32=basis32) as op:
        fs = [op.apply(dm.APPLY_A, torch.randn(3 * op.layout(0)["P"], dtype=torch.float64,
                                               generator=torch.Generator().manual_seed(q)).cuda(), op.face_tensor())
              for q in range(nb)]
        xs = [op.face_tensor() for _ in fs]
        infos = op.solve_block(fs, xs, mode=m, rtol=rtol, maxit=200)
        columns = min(i["iterations"] for i in infos)
        if crosses == "columns":
            assert columns > 40
        else:   # each column holds at least the active faces
            assert nb * columns * op.layout(0)["active_faces"] * (4 if basis32 else 8) > 128 << 20
            assert columns <= 32
        for f, x, info in zip(fs, xs, infos):
            alone = [op.face_tensor()]
            one = op.solve_block([f], alone, mode=m, rtol=rtol, maxit=200)[0]
            assert (info["status"], info["iterations"]) == (0, one["iterations"])
            assert float((x - alone[0]).norm()) <= 1e-12 * float(alone[0].norm())
