"""Meshes whose share of a block, with one more thing kept in LDS (pair
partials, element records, or all element terms in one chunk), comes within
2 KiB of what the kernel's static arrays leave: they take the next layout, and
the persistent kernel runs.  Against the per-iteration launches."""
import numpy as np
import pytest

import scenes
from helpers import make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,precision,model", [
    ((28, 14, 14), 0, "nh"), ((34, 13, 13), 0, "snh"), ((21, 18, 18), 0, "nh"), ((50, 14, 14), 0, "nh"),
    ((55, 16, 16), 0, "nh"), ((54, 15, 15), 1, "nh"), ((30, 18, 18), 0, "fcr"), ((61, 16, 16), 1, "fcr")])
def test_layouts_at_the_limit(dims, precision, model):
    sc = scenes.diff_bar_scene(seed=4, nx=dims[0], ny=dims[1], nz=dims[2], dx=0.01, lift=5e-4)
    v0 = 0.05 * np.sin(sc.X @ np.random.default_rng(1).uniform(5.0, 20.0, (3, 3)))
    out = []
    for profiled in (0, 1):
        ctx = make_ctx(sc, precision, iter_max=6, eps=0.0, term="delta_e", model=model)
        ctx.pncg_set_profiling(profiled)
        out.append(ctx.pncg_step(sc.X, v0, sc.h))
        assert ctx.pncg_get_persistent() == (1 - profiled, 0)
        ctx.close()
    assert out[0][2] == out[1][2]
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
