"""V-cycles on vectors outside the device's own memory: pageable and pinned
host tensors as input, as output and mixed with device ones give the values
of device tensors, bit for bit, for the single, block and batched V-cycle and
with symmetry planes."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

PLACES = {
    "device": lambda v: v.cuda(),
    "pageable": lambda v: v.clone(),
    "pinned": lambda v: torch.empty_like(v, pin_memory=True).copy_(v),
}


def inputs(op, count, dtype):
    """Random vectors on the active faces, on the host."""
    from paper_1301_3794_amd import dm
    n = 3 * op.layout(0)["P"]
    rnd = [torch.randn(n, dtype=torch.float64, generator=torch.Generator().manual_seed(q)) for q in range(count)]
    return [op.apply(dm.APPLY_A, v.cuda(), op.face_tensor()).to(dtype).cpu() for v in rnd]


@pytest.mark.parametrize("src,dst", [("pageable", "pageable"), ("pinned", "device"), ("device", "pageable")])
@pytest.mark.parametrize("planes", [False, True])
def test_vcycles(src, dst, planes):
    from paper_1301_3794_amd import dm
    geom = dm.ellipsoid((0.5 * (not planes),) * 3, (0.42, 0.45, 0.4))
    if planes:
        geom.bc_lo[:] = [dm.BC_PMC] * 3
    print(f"[case] vectors from {src} to {dst}, planes {planes}", flush=True)
    with dm.Operator(geom, (16, 16, 16), 1.0 / 16, 2.0) as op:
        for dt in (torch.float64, torch.float32):
            f = inputs(op, 3, dt)
            zero = torch.zeros_like(f[0])
            want = [op.vcycle(v.cuda(), zero.cuda()).cpu() for v in f]
            assert float(want[0].abs().max()) > 0
            got = op.vcycle(PLACES[src](f[0]), PLACES[dst](zero))
            assert torch.equal(got.cpu(), want[0])
            want = [x.cpu() for x in op.vcycle_block([v.cuda() for v in f], [zero.cuda() for _ in f])]
            # the first vector elsewhere, the others on the device
            ins = [PLACES[src if q == 0 else "device"](v) for q, v in enumerate(f)]
            outs = [PLACES[dst if q == 0 else "device"](zero) for q in range(3)]
            for x, ref in zip(op.vcycle_block(ins, outs), want):
                assert torch.equal(x.cpu(), ref)


@pytest.mark.parametrize("src,dst", [("pageable", "pageable"), ("pinned", "device"), ("device", "pageable")])
def test_batch(src, dst):
    from paper_1301_3794_amd import dm
    print(f"[case] batch vectors from {src} to {dst}", flush=True)
    geoms = [dm.ellipsoid((0.5, 0.5, 0.5), (0.4, 0.44, 0.47)), dm.sphere((0.5, 0.5, 0.5), 0.45)]
    b = dm.Batch(geoms, [(16, 16, 16), (8, 8, 8)], [1.0 / 16, 1.0 / 8], 5.0)
    try:
        f = [inputs(m, 1, torch.float32)[0] for m in b.members]
        want = [x.cpu() for x in b.vcycle([v.cuda() for v in f], [torch.zeros_like(v).cuda() for v in f])]
        got = b.vcycle([PLACES[src](v) for v in f], [PLACES[dst](torch.zeros_like(v)) for v in f])
        for x, ref in zip(got, want):
            assert float(ref.abs().max()) > 0 and torch.equal(x.cpu(), ref)
    finally:
        b.close()
