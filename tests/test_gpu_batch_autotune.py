"""The batch's autotuner times steps that follow one another, as a run takes
them, and reports errors of the caller's state alone."""
import numpy as np
import pytest

import scenes
from test_gpu_batch import _make_batch, _small_batch

pytestmark = pytest.mark.gpu


def _falling(scs, height):
    """Every scene at rest, height above its floor."""
    x = np.concatenate([s.x0 - [0.0, 0.0, s.x0[:, 2].min() - height] for s in scs])
    return x, np.zeros_like(x)


def test_timed_steps_follow_one_another():
    """4 mm above the floor a first step of 1/60 s falls free (2.7 mm), the
    second meets the floor and takes many more iterations.  The iterations
    summed over the timed steps are those of three steps in a row in each of
    the twelve settings (and of one step at the end), not of three first ones;
    the settings differ by the order of their sums only, so the comparison is
    with the nearer of the two."""
    import torch
    scs = _small_batch()
    bt, _ = _make_batch(scs, 0, 100, 1e-3, "delta_e")
    h = scs[0].h
    x, v = (torch.tensor(a, dtype=torch.float64, device="cuda:0") for a in _falling(scs, 4e-3))
    states, counts = [(x, v)], []
    for _ in range(3):
        xo, vo = torch.empty_like(x), torch.empty_like(v)
        bt.pncg_batch_step(*states[-1], h, xo, vo)
        counts.append(bt.pncg_batch_stats()[0].astype(np.int64).sum())
        states.append((xo, vo))
    t0 = bt.pncg_batch_stats()[2].sum()
    bt.pncg_batch_autotune(x, v, h, 2)
    iters, _, tot = bt.pncg_batch_stats()
    taken = tot.sum() - t0
    chain, repeat = 12 * sum(counts) + counts[0], 12 * 3 * counts[0]
    assert chain > 1.25 * repeat, (counts, chain, repeat)
    assert abs(taken - chain) < 0.1 * abs(chain - repeat), (taken, chain, repeat)
    # the statistics left are those of a step from the caller's state
    assert iters.astype(np.int64).sum() == counts[0]


def test_state_behind_its_floor_is_refused_and_leaves_nothing():
    import torch
    import paper_2405_08001_amd as P
    scs = _small_batch()
    bt, _ = _make_batch(scs, 0, 3, 0.0, "delta_e")
    h = scs[0].h
    x, v = (torch.tensor(a, dtype=torch.float64, device="cuda:0") for a in _falling(scs, 4e-3))
    below = x.clone()
    below[:, 2] -= 5e-3
    with pytest.raises(P.PncgError) as e:
        bt.pncg_batch_autotune(below, v, h, 1)
    assert e.value.code == -5
    bt.pncg_batch_autotune(x, v, h, 1)
