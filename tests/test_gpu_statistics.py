"""The statistics kernel's ways through a tally: planes (deposit cache) and a
row of groups per voxel (no cache), up to 16 groups and up to 64, rows read by
their own lanes (up to 12 groups) or by 16 lanes together, on grids that do not
fill its 16 x 16 tiles.  The same histories leave the same groups on both, so
dose (1e-11 of the maximum) and variance (a difference of group sums, 1e-9)
agree to the order of FP64 sums, LET_d as a ratio of such sums in voxels above
1% of the maximum dose (1e-9)."""
import numpy as np
import pytest

from test_gpu_tally_lines import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [3, 12, 13, 16, 17, 32, 33, 64])
@pytest.mark.parametrize("shape,mode", [((17, 3, 33), "dose"), ((31, 2, 15), "let")])
def test_rows_and_planes_of_groups(shape, mode, k):
    print("case: statistics", shape, mode, k, flush=True)
    d0, v0, l0, s0 = _run(shape, k, -1, mode)
    d1, v1, l1, s1 = _run(shape, k, 0, mode)
    assert s0["cache_slots"] == 0 and s1["cache_slots"] > 0
    assert s0["steps"] == s1["steps"] and d0.max() > 0.0
    np.testing.assert_allclose(d1, d0, rtol=0, atol=1e-11 * d0.max())
    np.testing.assert_allclose(v1, v0, rtol=0, atol=1e-9 * v0.max())
    np.testing.assert_allclose(s0["deposited"], s1["deposited"], rtol=1e-12)
    if mode == "let":
        hot = d0 > 0.01 * d0.max()
        assert hot.sum() > 20
        np.testing.assert_allclose(l1[hot], l0[hot], rtol=1e-9)
