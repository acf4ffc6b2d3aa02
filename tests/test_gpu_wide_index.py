"""Grids past the 24-bit column limit take the transport's 64-bit indices: the
histories of a beam near the low corner of a very long grid are those of the
same beam in a short one (same voxel size, so the same coordinates), and no
proton of 60 MeV reaches the short grid's far side.  Doses then agree to the
order of FP64 sums (1e-11 of the maximum), LET_d to the FP32 partial sums of
its numerator (1e-5)."""
import numpy as np
import pytest

from paper_1409_8336_amd import pmc, synth

pytestmark = pytest.mark.gpu

NY, NZ = 64, 8
VOXEL = (20.0, 0.2, 1.6)


def _run(mode, ny):
    import torch
    e = pmc.Engine(0, k_batches=2)
    e.load_physics(synth.nuclear_data())
    hu = synth.water_phantom(1, ny, NZ)
    e.load_geometry(hu, VOXEL, synth.material_table())
    sp = synth.pencil_spot(10.0, 0.1 * NY, 60.0)
    d = torch.zeros(hu.shape, dtype=torch.float64, device="cuda")
    if mode == "plans":
        slot = pmc.pmc_load_geometry_slot(e.ctx, hu[:, :NY].copy(), VOXEL, synth.material_table())
        d2 = torch.zeros((NZ, NY, 1), dtype=torch.float64, device="cuda")
        s = pmc.pmc_run_plans(e.ctx, [dict(geometry_id=0, spots=sp, n_histories=4000, d_dose=d),
                                      dict(geometry_id=slot, spots=sp, n_histories=500, d_dose=d2)], 7)
        s, extra = s[0], d2.cpu().numpy()
    elif mode == "let":
        let = torch.zeros_like(d)
        s = e.run_spots_let_dev(sp, 4000, 7, d, let)
        extra = let[:, :NY].cpu().numpy()
    else:
        s, extra = e.run_spots_dev(sp, 4000, 7, d), np.zeros(1)
    torch.cuda.synchronize()
    beyond = float(d[:, NY:].sum())
    out = d[:, :NY].cpu().numpy(), extra, beyond, s
    e.close()
    return out


@pytest.mark.parametrize("mode", ["dose", "let", "plans"])
def test_long_grid_equals_short_grid(mode):
    print("case:", mode, flush=True)
    short, short_x, _, ss = _run(mode, NY)
    wide, wide_x, beyond, sw = _run(mode, (1 << 24) + 1)
    assert beyond == 0.0 and short.max() > 0.0
    np.testing.assert_allclose(wide, short, rtol=0, atol=1e-11 * short.max())
    tol = 1e-5 if mode == "let" else 1e-11
    np.testing.assert_allclose(wide_x, short_x, rtol=0, atol=tol * (short_x.max() + 1e-300))
    for key in ("steps", "n_elastic", "n_nonelastic", "tally_atomics", "secondaries", "histories"):
        assert sw[key] == ss[key], key
