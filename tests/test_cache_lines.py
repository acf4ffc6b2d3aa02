"""The deposit cache's lines in the launch layout, checked on the CPU through
the C ABI (pmc_plan_cache, pmc_plan_launch): the regions the kernel indexes --
lines of eight sums, as many LET_d numerators, a key per line -- inside the
cache's memory, aligned, disjoint, and as many lines as fit it."""
import ctypes as C
import itertools

import pytest

from paper_1409_8336_amd import pmc


def _query(**kw):
    q = dict(block_threads=1024, grid_blocks=256, n_plans=1, batched=0, score_let=0, k_batches=10, n_mat=8,
             tally_cache=0, local_queue=0, n_spots=10, queue_capacity=0, n_histories=10 ** 6,
             max_plan_histories=10 ** 6, max_nvox=10 ** 6)
    q.update(kw)
    return q


@pytest.mark.parametrize("batched,let", itertools.product([0, 1], [0, 1]))
def test_lines_fill_the_cache_memory(batched, let):
    for block, n_mat, n_plans, cache in itertools.product([64, 256, 512, 1024], [1, 8, 16], [1, 64],
                                                          [0, -1, 512, 1000, 4097]):
        if n_plans > 1 and not batched:
            continue
        q = _query(block_threads=block, n_mat=n_mat, n_plans=n_plans, batched=batched, score_let=let, tally_cache=cache)
        rc, o, why = pmc.pmc_plan_launch(**q)
        rc2, c = pmc.pmc_plan_cache(**q)
        assert rc2 == rc, (q, why)
        if rc:
            continue
        if o["cache_slots"] == 0:
            assert c["lines"] == 0
            continue
        n = c["lines"]
        assert 1 <= n < 1 << 14 and c["line_sums"] == 8
        assert c["key_words"] == (2 if batched else 1)   # plan << 32 | line
        # words: begin, end, alignment in bytes
        sums = (c["sums_off"], c["sums_off"] + 2 * 8 * n, 8)
        nums = (c["num_off"], c["num_off"] + (2 * 8 * n if let else 0), 8)
        keys = (c["key_off"], c["key_off"] + c["key_words"] * n, 4 * c["key_words"])
        end = o["cache_off"]
        for b, e, al in (sums, nums, keys):
            assert b >= end and 4 * b % al == 0, (q, c)
            end = e
        assert end <= o["ctl_off"]
        assert 4 * o["ctl_off"] % 8 == 0   # the claims among the control words are 64-bit
        # no room for another line in the slots' memory
        slot_words = 2 + c["key_words"] + let
        line_words = 2 * 8 * (2 if let else 1) + c["key_words"]
        assert (n + 1) * line_words > o["cache_slots"] * slot_words


def test_refused_launches_have_no_cache_layout():
    out = pmc.pmc_cache_layout()
    assert pmc.lib().pmc_plan_cache(None, C.byref(out)) == pmc.PMC_ERR_ARG
    q = pmc.pmc_launch_query(**_query())
    assert pmc.lib().pmc_plan_cache(C.byref(q), None) == pmc.PMC_ERR_ARG
    for bad in (dict(block_threads=96), dict(tally_cache=16384), dict(n_mat=17), dict(max_nvox=0)):
        rc, _ = pmc.pmc_plan_cache(**_query(**bad))
        assert rc == pmc.PMC_ERR_ARG, bad


def test_no_lines_where_keys_do_not_fit():
    rc, c = pmc.pmc_plan_cache(**_query(max_nvox=400_000_000, k_batches=12))
    assert rc == pmc.PMC_OK and c["lines"] == 0
