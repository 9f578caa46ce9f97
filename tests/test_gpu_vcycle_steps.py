"""The V-cycle against its own steps, bit for bit.

A level's sweeps run as launches or, where it is small, whole in LDS; its
residual walks runs of the rows holding an active face or the whole grid by
class bytes; a block shares launches between vectors.  None of these choices
may change a value.  Two-level V-cycles with nu_pre = a and nu_post = b,
V(a, b), are taken apart with public calls:

    V(a, 0) f = s + V(0, 0) (f - M s)   with s = a sweeps from zero
    V(a, b) f = b reversed sweeps from V(a, 0) f

smooth() always launches its class updates and residual() walks the whole
grid, so every equality has the two forms on its sides.  Grids on either side
of the LDS rule, rows of one to many runs, with and without symmetry planes.

A batch picks LDS or launches for all its members at once: a member's values
may not depend on its companions.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIGMA = 2.0


def ellipsoid(n, r, planes):
    """An ellipsoid of semi-axes r times the box sides, centred in the box or, along an axis of symmetry, in the
    plane (the semi-axis then twice as long)."""
    from paper_1301_3794_amd import dm
    h = 1.0 / max(n)
    g = dm.ellipsoid([0.0 if p else 0.5 * m * h for m, p in zip(n, planes)],
                     [(2.0 if p else 1.0) * r * m * h for m, p in zip(n, planes)])
    g.bc_lo[:] = [dm.BC_PMC if p else dm.BC_PEC for p in planes]
    return g, h


CASES = [((16, 14, 10), 0.75), ((16, 16, 16), 0.47), ((18, 16, 12), 0.75), ((18, 18, 12), 0.75), ((24, 24, 24), 0.33),
         ((6, 10, 40), 0.46), ((34, 12, 10), 0.46), ((66, 10, 8), 0.6), ((130, 6, 4), 0.9)]


@pytest.mark.parametrize("planes", [(0, 0, 0), (1, 1, 0), (1, 1, 1)])
@pytest.mark.parametrize("n,r", CASES)
def test_vcycle_is_its_steps(n, r, planes):
    from paper_1301_3794_amd import dm
    print("[case]", n, r, planes, flush=True)
    geom, h = ellipsoid(n, r, planes)
    ops = {nu: dm.Operator(geom, n, h, SIGMA, levels=2, nu_pre=nu[0], nu_post=nu[1]) for nu in ((0, 0), (2, 0), (2, 3))}
    try:
        op = ops[2, 3]
        for dt in (torch.float64, torch.float32):
            new = lambda: op.face_tensor(dtype=dt)  # noqa: E731
            fs = [op.apply(dm.APPLY_A, torch.randn(3 * op.layout(0)["P"], dtype=torch.float64,
                                                   generator=torch.Generator().manual_seed(q)).cuda(),
                           op.face_tensor()).to(dt) for q in range(3)]
            want = []
            for f in fs:
                s = op.smooth(f, new(), sweeps=2)
                v20 = s + ops[0, 0].vcycle(op.residual(f, s, new()), new())
                assert float(v20.abs().max()) > 0
                # the padding of a face vector holds ghost images that a sum does not keep up to date
                inside = lambda v: v.reshape(3, n[2] + 2, n[1] + 2, n[0] + 2)[:, 1:-1, 1:-1, 1:-1]  # noqa: E731
                got = ops[2, 0].vcycle(f, new())
                assert torch.equal(inside(got), inside(v20)), "first sweeps and correction"
                want.append(inside(op.smooth(f, got.clone(), sweeps=3, reverse=True)).clone())
                assert torch.equal(inside(op.vcycle(f, new())), want[-1]), "last sweeps"
            for x, ref in zip(op.vcycle_block(fs, [new() for _ in fs]), want):
                assert torch.equal(inside(x), ref), "block"
    finally:
        for o in ops.values():
            o.close()


def test_batch_member_whatever_its_companions():
    from paper_1301_3794_amd import dm
    grids = [16, 40, 24]   # the first two depths of 16^3 fit LDS, those of 40^3 do not
    geoms = [dm.ellipsoid((0.5, 0.5, 0.5), s) for s in ((0.42, 0.36, 0.31), (0.33, 0.44, 0.38), (0.45, 0.3, 0.4))]
    print("[case] batches of", grids, flush=True)

    def run(pick):
        b = dm.Batch([geoms[q] for q in pick], [(grids[q],) * 3 for q in pick], [1.0 / grids[q] for q in pick], 5.0)
        try:
            f = [m.apply(dm.APPLY_A, torch.randn(3 * m.layout(0)["P"], dtype=torch.float64,
                                                 generator=torch.Generator().manual_seed(q)).cuda(),
                         m.face_tensor()).float() for q, m in zip(pick, b.members)]
            return dict(zip(pick, [x.clone() for x in b.vcycle(f, [torch.zeros_like(v) for v in f])]))
        finally:
            b.close()

    together = run([0, 1, 2])
    for q in range(3):
        alone = run([q])[q]
        assert float(alone.abs().max()) > 0
        assert torch.equal(together[q], alone), grids[q]
