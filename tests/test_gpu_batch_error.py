"""How far the fused FP32 V-cycle of a batch is from 64 bits.

Eight ellipsoids on 16^3 to 64^3 grids, smooth fields (the eigensolver's) and
random ones, four of each; the statistic is the geometric mean over fields and
members of the relative 2-norm error against the member's FP64 V-cycle (itself
within 1e-12 of the oracle, see test_gpu_parity.py).  The bounds are what rows
formed in FP32 from the FP32 fractions gave here, BOUND, plus 5% for another
order of sums; FP32 weights tabulated per row gave AFTER.
"""
import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BOUND = {"smooth": 5.096e-8, "random": 6.795e-8}
AFTER = {"smooth": 6.482e-8, "random": 7.607e-8}

NS = [16, 24, 32, 40, 48, 64, 32, 64]
SEMI = [(0.42, 0.36, 0.31), (0.33, 0.44, 0.38), (0.45, 0.3, 0.4), (0.37, 0.41, 0.46), (0.31, 0.47, 0.35),
        (0.44, 0.39, 0.42), (0.36, 0.33, 0.48), (0.47, 0.35, 0.38)]


def field(op, kind, seed):
    """An FP32 field on the active faces of a member."""
    n = op.dims[0]
    act = torch.from_numpy(op.fractions(0).reshape(7, -1)[:3].copy()).reshape(3, n + 2, n + 2, n + 2) > 0
    v = torch.zeros(act.shape, dtype=torch.float64)
    g = torch.Generator().manual_seed(seed)
    if kind == "random":
        v = torch.randn(v.shape, dtype=torch.float64, generator=g)
    else:
        x = torch.linspace(0, math.pi, n + 2, dtype=torch.float64)
        for c in range(3):
            a = float(torch.randn(1, generator=g))
            v[c] = a * torch.sin((1 + seed % 2) * x + c)[:, None, None] * torch.cos(x)[None, :, None] * \
                torch.sin(x + 0.3)[None, None, :]
    own = torch.zeros_like(v)
    own[:, 1:-1, 1:-1, 1:-1] = (v * act)[:, 1:-1, 1:-1, 1:-1]
    return own.float().reshape(-1).cuda()


def mean_error(dm, kind):
    b = dm.Batch([dm.ellipsoid((0.5, 0.5, 0.5), s) for s in SEMI], [(n,) * 3 for n in NS], [1.0 / n for n in NS], 5.0)
    try:
        logs = []
        for q in range(4):
            f = [field(m, kind, 100 * q + i) for i, m in enumerate(b.members)]
            ref = [m.vcycle(v.double(), m.face_tensor()).clone() for m, v in zip(b.members, f)]
            for x, r in zip(b.vcycle(f, [torch.zeros_like(v) for v in f]), ref):
                logs.append(math.log(float((x.double() - r).norm() / r.norm())))
        return math.exp(sum(logs) / len(logs))
    finally:
        b.close()


@pytest.mark.parametrize("kind", ["smooth", "random"])
def test_error_no_larger_than_from_the_fractions(kind):
    from paper_1301_3794_amd import dm
    print("[case] batch error", kind, flush=True)
    assert mean_error(dm, kind) <= 1.05 * BOUND[kind]
