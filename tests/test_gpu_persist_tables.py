"""Where the persistent kernels' tables come from: the first step or adjoint
that can use them, and nothing else.  A call without them launches per
iteration, with the same bits."""
import numpy as np
import pytest

import scenes
from helpers import make_ctx

pytestmark = pytest.mark.gpu

FIXED = dict(iter_max=8, eps=0.0, term="delta_e")


def _block(nx, ny, nz):
    sc = scenes.diff_bar_scene(seed=4, nx=nx, ny=ny, nz=nz, dx=0.01, lift=5e-4)
    return sc, 0.05 * np.sin(sc.X @ np.random.default_rng(1).uniform(5.0, 20.0, (3, 3)))


def _noalloc(ctx, sc, v0):
    import torch
    dev = torch.device("cuda:0")
    x, v = torch.tensor(sc.X, device=dev), torch.tensor(v0, device=dev)
    xo, vo = torch.empty_like(x), torch.empty_like(v)
    ctx.pncg_step_dev_noalloc(x, v, sc.h, xo, vo)
    return xo.cpu().numpy(), vo.cpu().numpy()


@pytest.mark.parametrize("precision", [0, 1])
def test_step_without_allocation_builds_none(precision):
    sc, v0 = _block(6, 5, 4)
    ctx = make_ctx(sc, precision, **FIXED)
    first = _noalloc(ctx, sc, v0)
    assert ctx.pncg_get_persistent() == (0, 0)
    second = ctx.pncg_step(sc.X, v0, sc.h)[:2]
    assert ctx.pncg_get_persistent() == (1, 0)
    third = _noalloc(ctx, sc, v0)
    assert ctx.pncg_get_persistent() == (2, 0)
    for a in (second, third):
        assert np.array_equal(first[0], a[0]) and np.array_equal(first[1], a[1])


def test_contexts_that_never_use_them():
    """Queries, the atomic scatter, the split step, a caller that profiles and
    dense contact from its first step on."""
    stack = scenes.small_contact_scene()
    v0 = np.zeros_like(stack.X)
    ctx = make_ctx(stack, 0, **FIXED)
    ctx.pncg_gradient(stack.X, stack.X, stack.h)
    ctx.pncg_hvp(stack.X, np.ones_like(stack.X), stack.h)
    assert ctx.pncg_get_persistent() == (0, 0)
    for _ in range(2):
        st = ctx.pncg_step(stack.X, v0, stack.h)[2]
        assert 4 * st["n_candidates"] > stack.nV
    assert ctx.pncg_get_persistent() == (0, 0)
    for kw in (dict(scatter=1), dict(split=True)):
        ctx = make_ctx(stack, 0, **kw, **FIXED)
        ctx.pncg_step(stack.X, v0, stack.h)
        assert ctx.pncg_get_persistent() == (0, 0)


def test_first_step_of_sparse_contact_and_a_new_mesh():
    pile = scenes.pile_scene(n_shapes=8, target_tets=12_000)
    small, vs = _block(6, 5, 4)
    ctx = make_ctx(pile, 0, **FIXED)
    other = make_ctx(pile, 0, **FIXED)
    other.pncg_set_profiling(1)
    a, b = [c.pncg_step(pile.x0, pile.v0, pile.h) for c in (ctx, other)]
    assert ctx.pncg_get_persistent()[0] > 0 and other.pncg_get_persistent() == (0, 0)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    # another mesh in the same context: its own tables, counts from zero
    for c in (ctx, other):
        c.pncg_set_mesh(small.X, small.tets, small.tris, small.edges, small.object_id)
        c.pncg_set_material(small.E, small.nu, small.rho)
        c.pncg_set_contact(small.dhat, small.kappa, small.cell, small.planes, 0)
    assert ctx.pncg_get_persistent() == (0, 0)
    a, b = [c.pncg_step(small.X, vs, small.h) for c in (ctx, other)]
    assert ctx.pncg_get_persistent() == (1, 0)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


def test_first_adjoint():
    sc, _ = _block(6, 5, 4)
    rng = np.random.default_rng(3)
    x = sc.X.copy()
    xbar, vbar = rng.standard_normal(x.shape), rng.standard_normal(x.shape)
    a, b = make_ctx(sc, 0), make_ctx(sc, 0)
    b.pncg_set_profiling(1)
    ra, rb = [c.pncg_adjoint_step(x, sc.h, xbar, vbar, cg_tol=0.0, cg_max=30) for c in (a, b)]
    assert a.pncg_get_persistent() == (1, 0) and b.pncg_get_persistent() == (0, 0)
    assert all(np.array_equal(p, q) for p, q in zip(ra[:3], rb[:3]))
    # the corotated product has no persistent kernel, and builds none
    c = make_ctx(sc, 0, model="fcr")
    c.pncg_adjoint_step(x, sc.h, xbar, vbar, cg_tol=0.0, cg_max=5)
    assert c.pncg_get_persistent() == (0, 0)
