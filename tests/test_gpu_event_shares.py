"""Cascade event lists of different lengths: a list that one workgroup per
compute unit holds is left to those, in even shares of the waves' lanes; a
longer one is worked by all workgroups.  Three plans in one launch (one list
with the events of all) against each plan alone (a list a third as long): the
same counts, doses to the order of FP64 sums (1e-11 of the maximum)."""
import numpy as np
import pytest

from paper_1409_8336_amd import pmc, synth
from parity_tools import ledger_residual

pytestmark = pytest.mark.gpu


# at 230 MeV three to four histories make an event: a few events, fewer than a
# tenth of the waves, about a share of 20 each, just above the events that one
# workgroup per unit holds (three plans only), well above
@pytest.mark.parametrize("n", [40, 300, 25_000, 90_000, 200_000])
def test_events_of_three_plans_in_one_list_equal_three_lists(n):
    import torch
    print("case: event shares, three plans of %d histories" % n, flush=True)
    hu = synth.water_phantom(24, 24, 90)
    spots = synth.pencil_spot(4.8, 4.8, 230.0, 0.3)
    e = pmc.Engine(0, flags=pmc.PMC_INC, block_threads=256, refill_lanes=16, batch_events=4)
    e.load_physics(synth.nuclear_data())
    e.load_geometry(hu, (0.4, 0.4, 0.4), synth.material_table())
    slots = [0] + [pmc.pmc_load_geometry_slot(e.ctx, hu, (0.4, 0.4, 0.4), synth.material_table()) for _ in range(2)]
    ds = [torch.zeros(hu.shape, dtype=torch.float64, device="cuda") for _ in range(3)]
    sums = pmc.pmc_run_plans(e.ctx, [dict(geometry_id=g, spots=spots, n_histories=n, d_dose=d)
                                      for g, d in zip(slots, ds)], 5)
    one = torch.zeros_like(ds[0])
    for p in range(3):
        s = e.run_spots_dev(spots, n, 5 + p, one)
        torch.cuda.synchronize()
        for key in ("steps", "n_nonelastic", "inc_events", "inc_secondaries", "inc_collisions"):
            assert sums[p][key] == s[key], (p, key, sums[p][key], s[key])
        assert s["inc_events"] == s["n_nonelastic"]
        assert ledger_residual(s) < 1e-5 and ledger_residual(sums[p]) < 1e-5
        want = one.cpu().numpy()
        np.testing.assert_allclose(ds[p].cpu().numpy(), want, rtol=0, atol=1e-11 * want.max())
    e.close()
