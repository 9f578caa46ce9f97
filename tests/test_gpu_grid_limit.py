"""The size limit of a grid: more than 2^31 - 1 padded elements are refused
(DM_EINVAL) before the fractions, which would take 7 arrays of that size, are
formed; a user geometry's are not read."""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("user", [False, True])
def test_grid_over_the_32_bit_limit(user):
    from paper_1301_3794_amd import dm
    n = (1290, 1290, 1290)   # 1292^3 = 2,156,689,088 padded elements
    assert (n[0] + 2) ** 3 > 2 ** 31 - 1
    print("[case] grid", n, "user fractions" if user else "sphere", flush=True)
    geom = dm.user_fractions(np.zeros((7, 8))) if user else dm.sphere()
    t0 = time.perf_counter()
    with pytest.raises(dm.DMError) as e:
        dm.Operator(geom, n, 1.0 / n[0], 1.0, levels=1)
    assert e.value.code == dm.DM_EINVAL and "too large" in str(e.value)
    assert time.perf_counter() - t0 < 20.0
