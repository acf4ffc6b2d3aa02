"""The deposit cache's 64-byte lines (eight tally elements along z, planes of
z-fastest elements) against a run without the cache (rows of groups, no lines),
on grids whose sides and planes do not fit the lines or the statistics'
16 x 16 tiles, with up to 16 groups and more: the same histories, so the same
counts and doses to the order of FP64 sums (1e-11 of the maximum; the variance,
a difference of group sums, to 1e-9), LET_d to the FP32 partial sums of its
numerator (1e-5)."""
import numpy as np
import pytest

from paper_1409_8336_amd import pmc, synth

pytestmark = pytest.mark.gpu

GRIDS = [(5, 3, 1), (3, 5, 7), (1, 1, 8), (17, 4, 9), (33, 2, 16), (16, 18, 47)]


def _run(shape, k, cache, mode):
    import torch
    nx, ny, nz = shape
    e = pmc.Engine(0, k_batches=k, block_threads=512, refill_lanes=8, batch_events=4, tally_cache=cache,
                   flags=pmc.PMC_INC if mode == "inc" else 0)
    e.load_physics(synth.nuclear_data())
    hu = (np.arange(nx * ny * nz, dtype=np.int64) * 37 % 900 - 300).astype(np.int16).reshape(nz, ny, nx)
    e.load_geometry(hu, (0.3, 0.3, 0.3), synth.material_table())
    sp = np.concatenate([synth.pencil_spot(0.15 * nx, 0.15 * ny, en, sigma_cm=0.1) for en in (70.0, 150.0)])
    d = torch.zeros(hu.shape, dtype=torch.float64, device="cuda")
    v, let = torch.zeros_like(d), torch.zeros_like(d)
    if mode == "let":
        s = e.run_spots_let_dev(sp, 6000, 3, d, let, v)
    else:
        s = e.run_spots_dev(sp, 6000, 3, d, v)
    torch.cuda.synchronize()
    e.close()
    return d.cpu().numpy(), v.cpu().numpy(), let.cpu().numpy(), s


@pytest.mark.parametrize("shape", GRIDS)
@pytest.mark.parametrize("mode,k", [("dose", 2), ("dose", 17), ("let", 10), ("inc", 16)])
def test_lines_equal_rows(shape, mode, k):
    print("case:", shape, mode, k, flush=True)
    d0, v0, l0, s0 = _run(shape, k, -1, mode)
    d1, v1, l1, s1 = _run(shape, k, 0, mode)
    assert s0["cache_slots"] == 0 and s1["cache_slots"] > 0
    for key in ("steps", "n_elastic", "n_nonelastic", "tally_atomics", "secondaries"):
        assert s0[key] == s1[key], key
    assert d0.max() > 0.0
    np.testing.assert_allclose(d1, d0, rtol=0, atol=1e-11 * d0.max())
    np.testing.assert_allclose(v1, v0, rtol=0, atol=1e-9 * v0.max())
    np.testing.assert_allclose(l1, l0, rtol=0, atol=1e-5 * max(l0.max(), 1e-300))
