"""An explicit list whose point-triangle pairs name interior vertices: steps
of several iterations against the per-iteration launches (which a context uses
while its profiling is on) and, in float64 and mixed, the float64 oracle.
Corners of pairs are read across blocks, so every vertex that a list may name
has to be kept where other blocks read it."""
import dataclasses

import numpy as np
import pytest

import scenes
from helpers import make_ctx, make_problem, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("where", ["interior", "mixed", "surface"])
def test_points_that_are_not_on_the_surface(where, precision):
    import paper_2405_08001_amd as L
    from oracle import pncg
    # every listed pair is active: the barrier reaches across the block, weakly
    sc = scenes.diff_bar_scene(seed=4, nx=9, ny=8, nz=7, dx=0.01, lift=0.01)
    sc = dataclasses.replace(sc, dhat=0.5, kappa=1e-4, self_contact=True, planes=np.zeros((0, 4)))
    rng = np.random.default_rng(6)
    surf = np.unique(sc.tris)
    inner = np.setdiff1d(np.arange(sc.nV), surf)
    assert len(inner) > 100
    points = {"interior": inner[::3], "surface": surf[::5], "mixed": np.concatenate([inner[::9], surf[::9]])}[where]
    pairs = np.stack([points, rng.integers(0, len(sc.tris), len(points))], axis=1)
    pairs = pairs[~(sc.tris[pairs[:, 1]] == pairs[:, :1]).any(axis=1)]
    none = np.zeros((0, 2), np.int64)
    v0 = 0.05 * np.sin(sc.X @ rng.uniform(5.0, 20.0, (3, 3)))
    out = []
    for profiled in (0, 1):
        ctx = make_ctx(sc, precision, iter_max=12, eps=0.0, term="delta_e", rest_exclude=False)
        ctx.pncg_set_profiling(profiled)
        ctx.pncg_set_candidates_override(L.KIND_PT, pairs)
        ctx.pncg_set_candidates_override(L.KIND_EE, none)
        x1, v1, s1 = ctx.pncg_step(sc.X, v0, sc.h)
        assert s1["n_active"] == len(pairs) and s1["iters"] == 12
        out.append((x1, v1) + ctx.pncg_step(x1, v1, sc.h)[:2])
        # without the list the same context goes back to the hash
        ctx.pncg_set_candidates_override(L.KIND_PT, None)
        ctx.pncg_set_contact(1e-3, 1e-4, 0.0, None, L.CONTACT_SELF)
        out[-1] += ctx.pncg_step(sc.X, v0, sc.h)[:2]
        ctx.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    P = make_problem(sc, rest_exclude=False)
    P.set_candidates_override(pairs, none)
    xo, _, st = pncg.step(P, sc.X, v0, sc.h, iter_max=12, eps=0.0, term="delta_e")
    print(f"{where} {precision}: {len(pairs)} pairs, against the oracle {rel(out[0][0] - sc.X, xo - sc.X):.1e}", flush=True)
    assert st.iters == 12
    assert rel(out[0][0] - sc.X, xo - sc.X) <= (1e-9 if precision == 0 else 1e-3)
