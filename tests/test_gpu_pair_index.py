"""The order of a vertex's pair entries: it depends on the set of pairs only,
whatever number of them one vertex has (the entries of up to 64 are ordered
from a wave's lanes, up to 256 from the wave's LDS, up to 1,024 from the
block's, more from memory) and in whatever order they come."""
import dataclasses

import numpy as np
import pytest

import scenes
from helpers import make_ctx, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 16, 63, 64, 65, 256, 257, 1024, 1025, 2000])
def test_entries_of_one_vertex(n):
    import paper_2405_08001_amd as L
    # every listed pair is active (the barrier reaches across the block, weakly)
    sc = scenes.diff_bar_scene(seed=4, nx=14, ny=14, nz=13, dx=0.01, lift=0.01)
    sc = dataclasses.replace(sc, dhat=0.5, kappa=1e-4, self_contact=True, planes=np.zeros((0, 4)))
    free = np.flatnonzero(~(sc.tris == 0).any(axis=1))
    assert len(free) >= 2000 and 0 in sc.tris
    pairs = np.stack([np.zeros(n, np.int64), free[:n]], axis=1)
    rng = np.random.default_rng(2)
    out = []
    for order, scatter in ((np.arange(n), 0), (rng.permutation(n), 0), (np.arange(n), 1)):
        ctx = make_ctx(sc, 0, iter_max=2, eps=0.0, term="delta_e", rest_exclude=False, scatter=scatter)
        ctx.pncg_set_candidates_override(L.KIND_PT, pairs[order])
        x, _, st = ctx.pncg_step(sc.X, np.zeros_like(sc.X), sc.h)
        assert st["n_active"] == n and st["iters"] == 2
        out.append(x)
    print(f"{n} pairs: segmented against atomic {rel(out[0] - sc.X, out[2] - sc.X):.1e}", flush=True)
    assert np.array_equal(out[0], out[1])
    assert rel(out[0], out[2]) <= 1e-12 and rel(out[0] - sc.X, out[2] - sc.X) <= 1e-9
