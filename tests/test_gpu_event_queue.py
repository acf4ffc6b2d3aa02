"""Nuclear events worked by full waves from the workgroups' event lists (runs
with at least two histories per lane) against events worked in place by the
waves that have them (the same histories on a larger grid of lanes): the same
counts, doses to the order of FP64 sums (1e-11 of the maximum), LET_d to the
FP32 partial sums of its numerator (1e-5)."""
import numpy as np
import pytest

from paper_1409_8336_amd import pmc, synth

pytestmark = pytest.mark.gpu


def _run(mode, n, **shape):
    import torch
    e = pmc.Engine(0, refill_lanes=8, flags=pmc.PMC_INC if mode == "inc" else 0, **shape)
    e.load_physics(synth.nuclear_data())
    hu = synth.ct_phantom(40, 36, 50, seed=4)
    e.load_geometry(hu, (0.4, 0.4, 0.4), synth.material_table())
    sp = synth.spot_field((8.0, 7.2), 2, 5, 90.0, 160.0, seed=2)
    d = torch.zeros(hu.shape, dtype=torch.float64, device="cuda")
    x = torch.zeros_like(d)
    if mode == "let":
        s = [e.run_spots_let_dev(sp, n, 9, d, x)]
    elif mode == "plans":
        hu2 = synth.ct_phantom(24, 20, 30, seed=6)
        slot = pmc.pmc_load_geometry_slot(e.ctx, hu2, (0.5, 0.5, 0.5), synth.material_table())
        x = torch.zeros(hu2.shape, dtype=torch.float64, device="cuda")
        s = pmc.pmc_run_plans(e.ctx, [dict(geometry_id=0, spots=sp, n_histories=n - n // 3, d_dose=d),
                                      dict(geometry_id=slot, spots=synth.pencil_spot(6.0, 5.0, 120.0),
                                           n_histories=n // 3, d_dose=x)], 9)
    else:
        s = [e.run_spots_dev(sp, n, 9, d)]
    torch.cuda.synchronize()
    e.close()
    return d.cpu().numpy(), x.cpu().numpy(), s


# workgroups of one wave, of several that are no power of two, of the largest
# size; few and many events a list, epochs shorter than the iterations a wave
# leaves out
@pytest.mark.parametrize("mode", ["dose", "let", "inc", "plans"])
@pytest.mark.parametrize("n,shape", [(40_000, dict(block_threads=64, blocks_per_cu=1, batch_events=1)),
                                     (110_000, dict(block_threads=192, blocks_per_cu=1, batch_events=8, epoch_steps=300)),
                                     (540_000, dict(block_threads=1024, batch_events=4, epoch_steps=2)),
                                     (540_000, dict(block_threads=1024, batch_events=4))])
def test_listed_events_equal_events_in_place(mode, n, shape):
    print("case:", mode, n, shape, flush=True)
    # in place (fewer than two histories a lane); a run too large for that against
    # the smallest workgroups, whose lists the first case checks
    ref = dict(block_threads=1024) if n < 524288 else dict(block_threads=64, blocks_per_cu=1)
    d0, x0, s0 = _run(mode, n, batch_events=4, tally_cache=-1, **ref)
    d1, x1, s1 = _run(mode, n, **shape)
    for a, b in zip(s0, s1):
        for key in ("steps", "n_elastic", "n_nonelastic", "tally_atomics", "histories"):
            assert a[key] == b[key], (key, a[key], b[key])
    assert sum(a["secondaries"] for a in s0[:1]) == sum(b["secondaries"] for b in s1[:1]) or mode == "plans"
    np.testing.assert_allclose(d1, d0, rtol=0, atol=1e-11 * d0.max())
    np.testing.assert_allclose(x1, x0, rtol=0, atol=(1e-5 if mode == "let" else 1e-11) * max(x0.max(), 1e-300))
