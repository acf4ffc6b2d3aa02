"""LET_d and batched secondaries at the accuracy their sums have.  LET_d
numerators and doses are FP64 sums on every way through the transport (deposit
cache or not, events listed or in place, 32- or 64-bit indices): in voxels above
1% of the largest dose, with up to 1e5 deposits each (1e-11) and a hundredfold
cancellation of the local part, LET_d agrees to 1e-9."""
import numpy as np
import pytest

import test_gpu_event_queue as events
import test_gpu_tally_lines as lines
import test_gpu_wide_index as wide

pytestmark = pytest.mark.gpu


def _same(let1, let0, dose0):
    hot = dose0 > 0.01 * dose0.max()
    assert hot.sum() > 0
    np.testing.assert_allclose(let1[hot], let0[hot], rtol=1e-9)


SHAPES = [(40_000, dict(block_threads=64, blocks_per_cu=1, batch_events=1)),
          (110_000, dict(block_threads=192, blocks_per_cu=1, batch_events=8, epoch_steps=300)),
          (540_000, dict(block_threads=1024, batch_events=4))]


def _in_place(mode, n):
    # fewer than two histories a lane; more than that: lists of the smallest workgroups
    ref = dict(block_threads=1024) if n < 524288 else dict(block_threads=64, blocks_per_cu=1)
    return events._run(mode, n, batch_events=4, tally_cache=-1, **ref)


@pytest.mark.parametrize("n,shape", SHAPES)
def test_listed_events(n, shape):
    print("case: LET_d, listed events", n, shape, flush=True)
    d0, x0, _ = _in_place("let", n)
    _, x1, _ = events._run("let", n, **shape)
    _same(x1, x0, d0)


@pytest.mark.parametrize("n,shape", SHAPES)
def test_secondaries_of_a_batch(n, shape):
    """A plan's secondaries are those its workgroups took plus all that passed
    through the shared queues: none of these with one generation, so the plans'
    numbers are the same."""
    print("case: secondaries of a batch", n, shape, flush=True)
    _, _, s0 = _in_place("plans", n)
    _, _, s1 = events._run("plans", n, **shape)
    assert all(s["generations"] == 1 for s in s0 + s1)
    assert [s["secondaries"] for s in s0] == [s["secondaries"] for s in s1]
    assert all(s["secondaries"] > 0 for s in s0)


@pytest.mark.parametrize("shape", [(17, 4, 9), (33, 2, 16), (16, 18, 47)])
def test_lines_and_rows(shape):
    print("case: LET_d, lines", shape, flush=True)
    d0, _, l0, _ = lines._run(shape, 10, -1, "let")
    _, _, l1, _ = lines._run(shape, 10, 0, "let")
    _same(l1, l0, d0)


def test_wide_indices():
    print("case: LET_d, wide indices", flush=True)
    d0, l0, _, _ = wide._run("let", wide.NY)
    _, l1, _, _ = wide._run("let", (1 << 24) + 1)
    _same(l1, l0, d0)
