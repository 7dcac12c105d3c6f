"""A persistent launch that gives up a wait (the host sets the limit so that
every launch does): the call starts again with a launch per iteration and has
that form's bits, from an intact state, in place, without allocation, on a
carried list and from a warm start; after 64 calls the persistent kernel runs
again.  The other side launches per iteration from the first (profiling on)."""
import numpy as np
import pytest

import scenes
from scenes import configs
from helpers import make_ctx

pytestmark = pytest.mark.gpu

AT_ONCE = -1


def _block(nx, ny, nz):
    sc = scenes.diff_bar_scene(seed=4, nx=nx, ny=ny, nz=nz, dx=0.01, lift=5e-4)
    return sc, 0.05 * np.sin(sc.X @ np.random.default_rng(1).uniform(5.0, 20.0, (3, 3)))


def _pair(sc, precision, **kw):
    out = []
    for profiled in (0, 1):
        ctx = make_ctx(sc, precision, **kw)
        ctx.pncg_set_profiling(profiled)
        out.append(ctx)
    return out


def _run(ctx, x0, v0, h, frames):
    import torch
    dev = torch.device("cuda:0")
    x, v = torch.tensor(x0, device=dev), torch.tensor(v0, device=dev)
    st, _ = ctx.pncg_run_dev(x, v, h, frames)
    return x.cpu().numpy(), v.cpu().numpy(), st


def _same(a, b):
    assert a[2] == b[2]
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    return a[0], a[1]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("dims", [(2, 2, 2), (13, 5, 4), (21, 16, 16)])
@pytest.mark.parametrize("model", ["nh", "fcr"])
def test_step_starts_again(dims, model, precision):
    sc, v0 = _block(*dims)
    a, b = _pair(sc, precision, iter_max=20, eps=0.0, term="delta_e", model=model)
    a.pncg_set_persistent(AT_ONCE)
    (xa, va, sa), (xb, vb, sb) = a.pncg_step(sc.X, v0, sc.h), b.pncg_step(sc.X, v0, sc.h)
    assert sa == sb and np.array_equal(xa, xb) and np.array_equal(va, vb)
    assert a.pncg_get_persistent() == (1, 1)
    # the next ones are launched per iteration at once
    _same(_run(a, xa, va, sc.h, 3), _run(b, xb, vb, sc.h, 3))
    assert a.pncg_get_persistent() == (1, 1) and b.pncg_get_persistent() == (0, 0)


@pytest.mark.parametrize("precision", [0, 1])
def test_run_in_place_and_after_the_back_off(precision):
    sc, v0 = _block(6, 5, 4)
    a, b = _pair(sc, precision, iter_max=6, eps=0.0, term="delta_e")
    a.pncg_set_persistent(AT_ONCE)
    x, v = _same(_run(a, sc.X, v0, sc.h, 2), _run(b, sc.X, v0, sc.h, 2))
    a.pncg_set_persistent(0)
    x, v = _same(_run(a, x, v, sc.h, 62), _run(b, x, v, sc.h, 62))
    assert a.pncg_get_persistent() == (1, 1)
    x, v = _same(_run(a, x, v, sc.h, 3), _run(b, x, v, sc.h, 3))
    assert a.pncg_get_persistent() == (4, 1)
    # and gives up once more
    a.pncg_set_persistent(AT_ONCE)
    _same(_run(a, x, v, sc.h, 2), _run(b, x, v, sc.h, 2))
    assert a.pncg_get_persistent() == (5, 2)


@pytest.mark.parametrize("precision", [0, 1])
def test_step_on_a_carried_list(precision):
    """The frame that starts again begins on the list of the frame before."""
    Xa, Ta = scenes.hex_grid(16, 16, 16, 0.01, origin=(0.0, 0.0, 5e-4))
    Xb, Tb = scenes.hex_grid(2, 2, 2, 0.01, origin=(0.073, 0.068, 0.1605 + 4e-4))
    X, tets, oid = scenes.merge_meshes([(Xa, Ta), (Xb, Tb)])
    sc = configs._scene(X, tets, E=2e5, nu=0.4, rho=1000.0, planes=[[0.0, 0.0, 1.0, 0.0]], dhat=1e-3, kappa=0.1,
                        h=1e-3, object_id=oid, self_contact=True)
    v0 = np.zeros_like(sc.X)
    v0[oid == 1, 2] = -0.1
    a, b = _pair(sc, precision, iter_max=25, eps=0.0, term="delta_e")
    _same(_run(a, sc.X, v0, sc.h, 1), _run(b, sc.X, v0, sc.h, 1))
    before = a.pncg_get_persistent()
    assert before[0] >= 1 and before[1] == 0
    a.pncg_set_persistent(AT_ONCE)
    # (the same state again: within the list that the first step left)
    ra, rb = _run(a, sc.X, v0, sc.h, 3), _run(b, sc.X, v0, sc.h, 3)
    assert rb[2][0]["rebuilds"] == 0 and rb[2][0]["n_active"] > 0
    _same(ra, rb)
    assert a.pncg_get_persistent() == (before[0] + 1, 1)


@pytest.mark.parametrize("precision", [0, 1])
def test_step_without_allocation(precision):
    import torch
    sc, v0 = _block(13, 5, 4)
    a, b = _pair(sc, precision, iter_max=20, eps=0.0, term="delta_e")
    x, v = _same(_run(a, sc.X, v0, sc.h, 1), _run(b, sc.X, v0, sc.h, 1))
    assert a.pncg_get_persistent() == (1, 0)
    a.pncg_set_persistent(AT_ONCE)
    dev = torch.device("cuda:0")
    xi, vi = torch.tensor(x, device=dev), torch.tensor(v, device=dev)
    st = a.pncg_step_dev_noalloc(xi, vi, sc.h, xi, vi)          # in place
    rb = _run(b, x, v, sc.h, 1)
    assert a.pncg_get_persistent() == (2, 1)
    assert st["iters"] == rb[2][0]["iters"] == 20
    assert np.array_equal(xi.cpu().numpy(), rb[0]) and np.array_equal(vi.cpu().numpy(), rb[1])


@pytest.mark.parametrize("warm", [False, True])
def test_adjoint_starts_again(warm):
    sc, _ = _block(12, 7, 6)
    rng = np.random.default_rng(3)
    x = sc.X.copy()
    x[:, 2] += 3e-4 - x[:, 2].min()
    xbar, vbar = rng.standard_normal(x.shape), rng.standard_normal(x.shape)
    a, b = _pair(sc, 0)
    kw = dict(cg_tol=1e-8, cg_max=20000)

    def both(s):
        ra, rb = [c.pncg_adjoint_step(x, sc.h, s * xbar, vbar, **kw) for c in (a, b)]
        assert ra[3] == rb[3] and all(np.array_equal(p, q) for p, q in zip(ra[:3], rb[:3]))
        return ra[3]

    for c in (a, b):
        c.pncg_set_adjoint_warm_start(warm)
    assert both(1.0)["cg_iters"] > 100 and a.pncg_get_persistent()[1] == 0
    n = a.pncg_get_persistent()[0]
    a.pncg_set_persistent(AT_ONCE)
    assert both(1.01)["cg_iters"] > 0
    assert a.pncg_get_persistent() == (n + 1, 1)
    assert both(1.02)["cg_iters"] > 0
    assert a.pncg_get_persistent() == (n + 1, 1)
