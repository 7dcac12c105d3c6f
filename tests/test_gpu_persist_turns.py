"""Contexts on threads of their own whose persistent launches do not fit on
the device together take turns: every call is a persistent one, no meeting
times out, and each gets the bits that it gets alone."""
import threading

import numpy as np
import pytest

import scenes
from helpers import make_ctx

pytestmark = pytest.mark.gpu


def _block(nx, ny, nz):
    sc = scenes.diff_bar_scene(seed=4, nx=nx, ny=ny, nz=nz, dx=0.01, lift=5e-4)
    return sc, 0.05 * np.sin(sc.X @ np.random.default_rng(1).uniform(5.0, 20.0, (3, 3)))


def _steps(dims, precision, n):
    sc, v = _block(*dims)
    ctx = make_ctx(sc, precision, iter_max=25, eps=0.0, term="delta_e")
    x, calls = sc.X, n
    for _ in range(n):
        x, v, _ = ctx.pncg_step(x, v, sc.h)
    return [x, v], ctx.pncg_get_persistent(), calls


def _adjoints(dims, n):
    sc, _ = _block(*dims)
    rng = np.random.default_rng(3)
    xbar, vbar = rng.standard_normal(sc.X.shape), rng.standard_normal(sc.X.shape)
    ctx = make_ctx(sc, 0)
    for _ in range(n):
        xbar, vbar, E, st = ctx.pncg_adjoint_step(sc.X, sc.h, xbar, vbar, cg_tol=0.0, cg_max=600)
        assert st["cg_iters"] == 600
    return [xbar, vbar, E], ctx.pncg_get_persistent(), 2 * n     # 512 iterations and the rest


def test_threads_take_turns():
    jobs = [lambda: _steps((40, 16, 16), 1, 12), lambda: _steps((6, 6, 6), 0, 40), lambda: _steps((50, 10, 10), 0, 12),
            lambda: _adjoints((30, 10, 10), 4)]
    alone = [j() for j in jobs]
    got = [None] * len(jobs)

    def work(i):
        got[i] = jobs[i]()

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for a, g in zip(alone, got):
        assert g is not None
        assert g[1] == a[1] == (a[2], 0)
        assert all(np.array_equal(p, q) for p, q in zip(a[0], g[0]))
