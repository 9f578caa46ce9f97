"""Which way a level's sweeps run, at the limits of the choice: a level on
either side of the face limits (6656 in FP64, 10240 in FP32) and of the LDS
size, as the finest level of a two-level V-cycle, one vector and a block; and
a batch of more members than one copy launch takes (64).

Tolerances (as in test_gpu_parity.py and test_gpu_batch.py): FP64 1e-12, FP32
5e-5 against the oracle; a member's own V-cycle 1e-6.
"""
import numpy as np
import pytest

from oracle import geometry as geo, multigrid as omg
import layout as lay

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def rel_inf(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


# (n, semi-axes over the box sides): active faces, 3 P values
@pytest.mark.parametrize("n,r", [
    ((16, 14, 10), 0.75),   # 6,196, 10,368: LDS in both precisions
    ((16, 14, 12), 0.75),   # 7,480, 12,096: past the FP64 face limit
    ((18, 16, 12), 0.75),   # 9,648, 15,120: the FP32 one just above
    ((18, 18, 12), 0.75),   # 10,884, 16,800: past the FP32 face limit
    ((20, 20, 20), 0.33),   # 4,500, 31,944: does not fit in FP64
    ((24, 24, 24), 0.33),   # 7,512, 52,728: does not fit in FP32 either
])
def test_vcycle_at_the_lds_limits(n, r):
    from paper_1301_3794_amd import dm
    h, sigma = 1.0 / max(n), 2.0
    fr = geo.fractions(geo.Ellipsoid(tuple(0.5 * h * m for m in n), tuple(r * h * m for m in n)), n, h)
    vc = omg.VCycle(fr, n, h, sigma, 2)
    L = vc.levels[0]
    print(f"[case] n={n} faces={L.op.act.size}", flush=True)
    fs = []
    for q in range(3):
        f = np.zeros(L.op.grid.n_faces)
        f[L.op.act] = np.random.default_rng(q).standard_normal(L.op.act.size)
        fs.append(f)
    with dm.Operator(dm.user_fractions(lay.fractions_to_padded(fr, n)), n, h, sigma, levels=2) as op:
        for dt, tol in ((torch.float64, 1e-12), (torch.float32, 5e-5)):
            fd = [torch.tensor(lay.faces_to_padded(f, n), dtype=dt, device="cuda") for f in fs]
            xs = [op.vcycle(fd[0], op.face_tensor(dtype=dt))]
            xs += op.vcycle_block(fd, [op.face_tensor(dtype=dt) for _ in fd])
            for f, x in zip([fs[0]] + fs, xs):
                assert rel_inf(lay.faces_from_padded(x.double().cpu().numpy(), n), vc(f)) <= tol


def test_batch_of_more_members_than_a_copy_launch_takes():
    from paper_1301_3794_amd import dm
    nb, n = 67, 8
    geoms = [dm.ellipsoid((0.5, 0.5, 0.5), (0.4 + 0.001 * q, 0.44, 0.47 - 0.001 * q)) for q in range(nb)]
    b = dm.Batch(geoms, [(n, n, n)] * nb, [1.0 / n] * nb, 5.0)
    print("[case] batch of", nb, flush=True)
    try:
        fs, refs = [], []
        for q, m in enumerate(b.members):
            v = torch.randn(3 * m.layout(0)["P"], dtype=torch.float64, generator=torch.Generator().manual_seed(q)).cuda()
            fs.append(m.apply(dm.APPLY_A, v, m.face_tensor()).float())
            refs.append(m.vcycle(fs[q].clone(), m.face_tensor(dtype=torch.float32)).clone())
        xs = [torch.zeros_like(f) for f in fs]
        b.vcycle(fs, xs)
        for x, ref in zip(xs, refs):
            scale = float(ref.abs().max())
            assert scale > 0
            assert float((x - ref).abs().max()) <= 1e-6 * scale
    finally:
        b.close()
