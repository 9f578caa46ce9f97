"""The rule that says which levels sweep in LDS, with the counts it decides by.

An iterate of 3 P values in at most 160 KB, and at most 6,656 active faces in
FP64, 10,240 in FP32, 8,000 in FP32 with symmetry planes.  Every case states
its faces and 3 P, so that a change of the fractions cannot move it to the
other side unseen.

  * without planes the path shows in a batch of one member: its fused V-cycle
    of two levels has 7 launches where the finer level sweeps in LDS and 29
    where each of the 24 classes is launched;
  * with planes the V-cycles on both sides of each limit are compared with the
    oracle, FP64 1e-12 and FP32 5e-5, as in test_gpu_pmc.py.
"""
import numpy as np
import pytest

from oracle import geometry as geo, symmetry as sym
import layout as lay

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

KB160 = 160 * 1024


def most(elem, planes):
    return 6656 if elem == 8 else 8000 if planes else 10240


@pytest.mark.parametrize("n,r,faces,three_p,in_lds", [
    ((16, 14, 10), 0.75, 6196, 10368, True),
    ((18, 16, 12), 0.75, 9648, 15120, True),
    ((18, 18, 12), 0.75, 10884, 16800, False),   # too many faces
    ((32, 32, 32), 0.20, 3948, 117912, False),   # few faces, does not fit
])
def test_path_of_a_batch(n, r, faces, three_p, in_lds):
    from paper_1301_3794_amd import dm
    h = 1.0 / max(n)
    geom = dm.ellipsoid([0.5 * v * h for v in n], [r * v * h for v in n])
    b = dm.Batch([geom], [n], [h], 2.0, levels=2)
    try:
        lay0 = b.members[0].layout(0)
        print("[case] batch of", n, lay0, flush=True)
        assert (lay0["active_faces"], 3 * lay0["P"]) == (faces, three_p)
        assert in_lds == (4 * three_p <= KB160 and faces <= most(4, False))
        assert b.stats()["launches_per_vcycle"] == (7 if in_lds else 29)
    finally:
        b.close()


@pytest.mark.parametrize("nh,faces,three_p,lds64,lds32", [
    ((16, 14, 10), 6478, 10368, True, True),
    ((14, 14, 12), 6842, 10752, False, True),
    ((16, 14, 12), 7822, 12096, False, True),
    ((14, 14, 14), 8018, 12288, False, False),
])
def test_vcycle_with_planes(nh, faces, three_p, lds64, lds32):
    from paper_1301_3794_amd import dm
    h, sigma = 1.0 / max(nh), 2.0
    nf = (2 * nh[0], 2 * nh[1], nh[2])
    fr = geo.fractions(geo.Ellipsoid([0.5 * v * h for v in nf], [0.75 * v * h for v in nf]), nf, h)
    vc = sym.HalfVCycle(fr, nh, h, sigma, (0, 1), 2)
    L = vc.levels[0]
    print("[case] planes", nh, L.op.act.size, flush=True)
    assert (L.op.act.size, 3 * lay.padded_size(nh)) == (faces, three_p)
    for elem, lds in ((8, lds64), (4, lds32)):
        assert lds == (elem * three_p <= KB160 and faces <= most(elem, True))
    geom = dm.user_fractions(lay.fractions_to_padded(vc.exts[0].half_fractions(fr), nh),
                             bc_lo=(dm.BC_PMC, dm.BC_PMC, dm.BC_PEC))
    fs = []
    for q in range(2):
        f = np.zeros(L.op.grid.n_faces)
        f[L.op.act] = np.random.default_rng(q).standard_normal(faces)
        fs.append(f)
    refs = [vc(f) for f in fs]
    with dm.Operator(geom, nh, h, sigma, levels=2) as op:
        assert op.layout(0)["active_faces"] == faces
        for dt, tol in ((torch.float64, 1e-12), (torch.float32, 5e-5)):
            fd = [torch.tensor(lay.faces_to_padded(f, nh), dtype=dt, device="cuda") for f in fs]
            xs = [op.vcycle(fd[0], op.face_tensor(dtype=dt))]
            xs += op.vcycle_block(fd, [op.face_tensor(dtype=dt) for _ in fd])
            for x, ref in zip(xs, [refs[0]] + refs):
                got = lay.faces_from_padded(x.double().cpu().numpy(), nh)
                assert np.max(np.abs(got - ref)) <= tol * np.max(np.abs(ref))
