"""LET_d through the deposit cache's lines against LET_d by atomics alone:
numerators and doses are FP64 sums on both ways, so LET_d agrees to the order
of sums: in voxels above 1% of the largest dose, with up to 1e4 deposits each
(1e-12) and a hundredfold cancellation of the local part, 1e-9."""
import numpy as np
import pytest

from paper_1409_8336_amd import pmc, synth

pytestmark = pytest.mark.gpu


def _let(n, **shape):
    import torch
    e = pmc.Engine(0, refill_lanes=8, batch_events=4, **shape)
    e.load_physics(synth.nuclear_data())
    hu = synth.ct_phantom(40, 36, 50, seed=4)
    e.load_geometry(hu, (0.4, 0.4, 0.4), synth.material_table())
    d = torch.zeros(hu.shape, dtype=torch.float64, device="cuda")
    x = torch.zeros_like(d)
    s = e.run_spots_let_dev(synth.pencil_spot(8.0, 7.2, 150.0, 0.3), n, 9, d, x)
    torch.cuda.synchronize()
    e.close()
    return d.cpu().numpy(), x.cpu().numpy(), s


# the fewest lines a launch may have, the automatic number; epochs as given by
# the run, and long enough to overflow the lines
@pytest.mark.parametrize("shape", [dict(block_threads=256, tally_cache=512), dict(block_threads=1024),
                                   dict(block_threads=1024, epoch_steps=64)])
def test_let_through_lines_equals_let_by_atomics(shape):
    print("case: LET_d sums", shape, flush=True)
    d0, x0, s0 = _let(100_000, block_threads=1024, tally_cache=-1)
    d1, x1, s1 = _let(100_000, **shape)
    assert s0["steps"] == s1["steps"] and s1["cache_slots"] > 0
    np.testing.assert_allclose(d1, d0, rtol=0, atol=1e-11 * d0.max())
    hot = d0 > 0.01 * d0.max()
    assert hot.sum() > 100
    np.testing.assert_allclose(x1[hot], x0[hot], rtol=1e-9)
