"""Scenes stepped by teams of workgroups, whose members exchange P g by words
(up to 512 vertices) or through the caches: on either side of that size, at the
two block sizes that read the partial sums differently, the steps repeat to the
bit, also after other scenes have used the team's buffers, and match the same
scenes on one workgroup each up to the order of the sums."""
import numpy as np
import pytest

import scenes
from helpers import rel
from test_gpu_batch import _make_batch, _states, _step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [256, 512])
@pytest.mark.parametrize("precision", [0, 1])
def test_teams_on_either_side_of_the_word_exchange(precision, block):
    # 425 and 729 vertices by teams, 20 and 208 on single workgroups
    scs = []
    for n in (7, 8, 2, 4, 7):
        scs += scenes.batched_scenes(seed=n, n_scenes=1, t_lo=6 * n ** 3, t_hi=6 * n ** 3 + 1)
    off = np.cumsum([0] + [s.nV for s in scs])
    assert min(s.nV for s in scs) < 512 < max(s.nV for s in scs)
    xs, vs = _states(scs, 8)
    x, v, h = np.concatenate(xs), np.concatenate(vs), scs[0].h
    bt, _ = _make_batch(scs, precision, 6, 0.0, "delta_e")
    bt.pncg_batch_set_block(block)
    res = {}
    for team in (1, 8):
        bt.pncg_batch_set_split(team)
        a = _step(bt, x, v, h)
        b = _step(bt, a[0], a[1], h)      # another step on the same buffers
        c = _step(bt, x, v, h)
        assert np.array_equal(a[0], c[0]) and np.array_equal(a[1], c[1])
        assert np.isfinite(b[0]).all()
        res[team] = (bt.pncg_batch_get_config()["teams"], a[0])
    assert res[8][0] < res[1][0]
    for i in range(len(scs)):
        p, q, r = [u[off[i]:off[i + 1]] for u in (res[8][1], res[1][1], x)]
        print(f"  scene {i}: {scs[i].nV} vertices {rel(p, q):.1e} {rel(p - r, q - r):.1e}", flush=True)
        assert rel(p, q) <= (1e-12 if precision == 0 else 1e-6)
        assert rel(p - r, q - r) <= (1e-9 if precision == 0 else 1e-3)
