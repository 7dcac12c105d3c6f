"""The persistent kernel of the adjoint's CG iterations against a launch per
iteration (which a context uses while its profiling is on): both sum in the
same order, so the adjoint has the same bits either way, for meshes of one or
more tets per thread and element chunks, across launches (one runs at most 512
iterations), for each way to stop, with a warm start and beside contact with
the floor."""
import numpy as np
import pytest

import scenes
from helpers import make_ctx

pytestmark = pytest.mark.gpu


def _case(dims, seed=3):
    sc = scenes.diff_bar_scene(seed=4, nx=dims[0], ny=dims[1], nz=dims[2], dx=0.01, lift=5e-4)
    rng = np.random.default_rng(seed)
    x = sc.X + 1e-4 * np.sin(50.0 * sc.X) @ rng.standard_normal((3, 3))
    x[:, 2] += 3e-4 - x[:, 2].min()          # the lowest vertices in the floor's barrier
    return sc, x, rng.standard_normal(x.shape), rng.standard_normal(x.shape)


def _pair(sc, model="nh", warm=False):
    out = []
    for profiled in (0, 1):
        ctx = make_ctx(sc, 0, model=model)
        ctx.pncg_set_profiling(profiled)
        ctx.pncg_set_adjoint_warm_start(warm)
        out.append(ctx)
    return out


def _same(ctxs, sc, x, xbar, vbar, **kw):
    a, b = [c.pncg_adjoint_step(x, sc.h, xbar, vbar, **kw) for c in ctxs]
    assert a[3] == b[3]
    for i in range(3):
        assert np.array_equal(a[i], b[i]) and np.isfinite(a[i]).all()
    return a[3]


# fewer blocks than compute units; one and two logical blocks to a workgroup;
# more tets than threads; two and three element chunks; too large for LDS
@pytest.mark.parametrize("dims", [(2, 2, 2), (13, 5, 4), (15, 14, 13), (50, 10, 10), (30, 20, 20), (50, 17, 17),
                                  (26, 26, 27), (45, 27, 26)])
def test_bits_over_sizes(dims):
    sc, x, xbar, vbar = _case(dims)
    st = _same(_pair(sc), sc, x, xbar, vbar, cg_tol=0.0, cg_max=25)
    assert st["cg_iters"] == 25 or dims == (2, 2, 2)


@pytest.mark.parametrize("model", ["nh", "snh", "arap", "fcr"])
def test_bits_over_materials(model):
    sc, x, xbar, vbar = _case((17, 9, 8))
    st = _same(_pair(sc, model), sc, x, xbar, vbar, cg_tol=1e-10, cg_max=20000)
    assert st["reason"] == 0 and st["cg_iters"] > 100


@pytest.mark.parametrize("cg_max", [1, 510, 511, 512, 513, 1100])
def test_bits_past_one_launch(cg_max):
    sc, x, xbar, vbar = _case((20, 9, 9))
    st = _same(_pair(sc), sc, x, xbar, vbar, cg_tol=0.0, cg_max=cg_max)
    assert st["cg_iters"] == cg_max and st["reason"] == 1


def test_bits_of_the_ends():
    """A right-hand side of zero, a tolerance that the start meets, and a warm
    start from the last solution (whose buffer changes with every solve)."""
    sc, x, xbar, vbar = _case((12, 7, 6))
    ctxs = _pair(sc, warm=True)
    z = np.zeros_like(x)
    assert _same(ctxs, sc, x, z, z, cg_tol=1e-10, cg_max=50)["cg_iters"] == 0
    first = _same(ctxs, sc, x, xbar, vbar, cg_tol=1e-8, cg_max=20000)
    again = _same(ctxs, sc, x, xbar, vbar, cg_tol=1e-7, cg_max=20000)
    third = _same(ctxs, sc, x, 1.01 * xbar, vbar, cg_tol=1e-8, cg_max=20000)
    assert first["cg_iters"] > 100 and again["cg_iters"] == 0 and 0 < third["cg_iters"]


def test_bits_beside_steps():
    """Steps and adjoints take turns on the same exchange buffers."""
    sc, x, xbar, vbar = _case((15, 14, 13))
    ctxs = _pair(sc)
    for c in ctxs:
        c.pncg_set_solver(20, 0.0, 0, sc.gravity, 0)
    v = np.zeros_like(x)
    for n in (7, 20, 21):
        (xa, va, sa), (xb, vb, sb) = [c.pncg_step(x, v, sc.h) for c in ctxs]
        assert sa == sb and np.array_equal(xa, xb)
        _same(ctxs, sc, xa, xbar, vbar, cg_tol=0.0, cg_max=n)
        x, v = xa, va


def test_indefinite_is_reported():
    """A block under strong compression, where H is indefinite: both forms end
    with the same error, and the contexts solve again afterwards."""
    import paper_2405_08001_amd as P
    sc, x, xbar, vbar = _case((6, 5, 4))
    ctxs = _pair(sc)
    squeezed = x * np.array([0.05, 1.0, 1.0])
    for c in ctxs:
        with pytest.raises(P.PncgError) as e:
            c.pncg_adjoint_step(squeezed, sc.h, xbar, vbar, cg_tol=1e-10, cg_max=1000)
        assert e.value.code == P.E_INDEFINITE
    _same(ctxs, sc, x, xbar, vbar, cg_tol=1e-10, cg_max=20000)
