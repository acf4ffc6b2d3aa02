"""Workgroup size of runs too small to be tuned, where the caller leaves it
open: large workgroups go with a deposit cache of many lines; without one (or
with one made small by the caller) runs keep the small workgroups."""
import pytest

from paper_1409_8336_amd import pmc, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,cache,let,lanes", [
    (39_000, 0, False, 256),
    (41_000, 0, False, 1024),
    (41_000, 0, True, 1024),
    (41_000, -1, False, 256),
    (41_000, -1, True, 256),
    (41_000, 512, False, 256),
    (41_000, 2048, True, 256),
    (41_000, 4096, True, 1024),
])
def test_workgroup_size_of_small_runs(n, cache, let, lanes):
    import torch
    print("case: small run", n, cache, let, flush=True)
    e = pmc.Engine(0, tally_cache=cache)
    e.load_physics(synth.nuclear_data())
    hu = synth.water_phantom(16, 16, 40)
    e.load_geometry(hu, (0.2, 0.2, 0.2), synth.material_table())
    d = torch.zeros(hu.shape, dtype=torch.float64, device="cuda")
    x = torch.zeros_like(d)
    sp = synth.pencil_spot(1.6, 1.6, 90.0)
    s = e.run_spots_let_dev(sp, n, 3, d, x) if let else e.run_spots_dev(sp, n, 3, d)
    e.close()
    assert s["block_threads"] == lanes
