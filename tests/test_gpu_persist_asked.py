"""Tables that only some of a mesh's callers can use: they are built for the
first that can, the others launch per iteration, and all have the bits of the
launches."""
import numpy as np
import pytest

import scenes
from helpers import make_ctx

pytestmark = pytest.mark.gpu


def _pair(nx, ny, nz):
    sc = scenes.diff_bar_scene(seed=4, nx=nx, ny=ny, nz=nz, dx=0.01, lift=5e-4)
    ctxs = [make_ctx(sc, 0, iter_max=4, eps=0.0, term="delta_e") for _ in range(2)]
    ctxs[1].pncg_set_profiling(1)       # launches only
    v0 = 0.05 * np.sin(sc.X @ np.random.default_rng(1).uniform(5.0, 20.0, (3, 3)))
    return sc, v0, ctxs


def _same(a, b):
    return all(np.array_equal(p, q) for p, q in zip(a, b) if isinstance(p, np.ndarray))


def test_eight_chunks_serve_the_adjoint_alone():
    """124,800 tets float64 fit in eight chunks of a block's waves, where a
    step gains nothing over its launches, and CG iterations do."""
    sc, v0, (ctx, ref) = _pair(32, 26, 25)
    bars = np.random.default_rng(3).standard_normal((2,) + sc.X.shape)
    step = [c.pncg_step(sc.X, v0, sc.h) for c in (ctx, ref)]
    assert ctx.pncg_get_persistent() == (0, 0) and _same(*step)
    adj = [c.pncg_adjoint_step(sc.X, sc.h, *bars, cg_tol=0.0, cg_max=8) for c in (ctx, ref)]
    assert ctx.pncg_get_persistent() == (1, 0) and _same(*adj)
    # with the tables there, steps still launch
    step = [c.pncg_step(sc.X, v0, sc.h) for c in (ctx, ref)]
    assert ctx.pncg_get_persistent() == (1, 0) and _same(*step)


def test_lanes_fit_where_tets_do_not():
    """131,712 tets float64: a share fits by (tet, corner) lane but not by tet,
    so the corotated model has tables and Neo-Hookean steps and adjoints none,
    whichever comes first."""
    sc, v0, (ctx, ref) = _pair(28, 28, 28)
    bars = np.random.default_rng(3).standard_normal((2,) + sc.X.shape)

    def both(model):
        for c in (ctx, ref):
            c.pncg_set_model(model)
        assert _same(*[c.pncg_step(sc.X, v0, sc.h) for c in (ctx, ref)])
        return ctx.pncg_get_persistent()

    assert both("nh") == (0, 0)
    ctx.pncg_adjoint_step(sc.X, sc.h, *bars, cg_tol=0.0, cg_max=4)
    assert ctx.pncg_get_persistent() == (0, 0)
    assert both("fcr") == (1, 0)
    assert both("nh") == (1, 0)
    assert both("arap") == (2, 0)
