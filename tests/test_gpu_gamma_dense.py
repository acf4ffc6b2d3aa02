"""Gamma index of regions where most voxels are above the cutoff: runs of 512
voxels with 256 and more evaluated ones take another course (a voxel per
lane) than the others.  Against the oracle, where a voxel settles at once,
within the first offsets, or searches the whole sphere, and where only some of
a run do.

Tolerance: a search point is an FP32 voxel coordinate, at most delta = 2^-23 n
from the oracle's on an axis of n voxels, and the interpolated dose changes by
at most 2 max(ev) per voxel and axis, so gamma moves by at most 6 max(ev) delta
/ (dose criterion), beside an FP32 result's 1e-5."""
import numpy as np
import pytest

from oracle import denoiser_oracle as D
from paper_1409_8336_amd import unet

pytestmark = pytest.mark.gpu

VOX = (0.23, 0.27, 0.31)   # no multiple of the step: no search point on a face


# voxels above the cutoff in each run of 512 (the last run is the grid's rest)
@pytest.mark.parametrize("shape,above", [
    ((4, 16, 16), (512, 512)),
    ((4, 16, 16), (256, 255)),     # just dense, just not
    ((1, 19, 27), (512, 1)),       # 513 voxels
    ((3, 13, 21), (300, 307)),     # 819: a dense last run of 307
])
@pytest.mark.parametrize("off,search", [
    ("near", 0.3), ("far", 0.3), ("far", 0.55), ("mixed", 0.3), ("mixed", 0.55), ("mixed", 0.0),
    ("far", 0.35), ("far", 0.357), ("mixed", 0.4),   # seven steps, the next shell, eight
])
def test_dense_runs_match_oracle(shape, above, off, search):
    import torch
    print("case: dense gamma", shape, above, off, search, flush=True)
    rng = np.random.default_rng(67)
    n = int(np.prod(shape))
    ref = np.full(n, 0.05)
    for run, k in enumerate(above):
        at = np.arange(512 * run, min(512 * (run + 1), n))
        ref[rng.choice(at, min(k, len(at)), replace=False)] = 1.0
    ref[ref == 1.0] = 1.0 + rng.random(int((ref == 1.0).sum()))
    ref[np.argmax(ref)] = 2.0
    factor = {"near": 1.005, "far": 3.0}.get(off)
    if factor is None:   # settled at once, soon, late
        factor = rng.choice((1.0, 1.02, 1.5, 3.0), n)
    ref = ref.reshape(shape)
    ev = ref * np.reshape(factor, shape if np.ndim(factor) else ())
    kw = dict(dose_frac=0.02, dta_cm=0.3, cutoff_frac=0.1, search_cm=search, step_cm=0.05)
    g_o, rate_o, n_o = D.gamma_index(ref, ev, VOX, **kw)
    gam = torch.zeros(shape, dtype=torch.float32, device="cuda")
    rate, count = unet.pmc_gamma_index(torch.from_numpy(ref).cuda(), torch.from_numpy(ev).cuda(), VOX, gamma=gam, **kw)
    g = gam.cpu().numpy().astype(np.float64)
    assert count == n_o == (ref > 0.2).sum()
    assert np.array_equal(g == -1.0, g_o < 0)
    bound = 1e-5 * np.maximum(1.0, g_o) + 6 * ev.max() / (0.02 * ref.max()) * 2.0 ** -23 * max(shape)
    assert np.all((np.abs(g - g_o) <= bound)[g_o >= 0])
    amb = int(((g_o >= 0) & (np.abs(g_o - 1.0) <= bound)).sum())
    assert abs(rate - rate_o) <= amb / max(n_o, 1) + 1e-12
