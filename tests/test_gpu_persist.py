"""The persistent iteration kernel against the per-iteration launches (which
a context uses while its profiling is on): both sum in the same order, so a
step has the same bits either way, whatever the mesh size (one or two logical
blocks in a workgroup, a few workgroups or one per compute unit, remainders of
every slice), material, precision, stop rule and contact, across list rebuilds
and across launches (a launch runs at most 512 iterations)."""
import numpy as np
import pytest

import scenes
from helpers import make_ctx

pytestmark = pytest.mark.gpu


def _run(sc, x0, v0, frames, profiled, precision, **kw):
    import torch
    dev = torch.device("cuda:0")
    ctx = make_ctx(sc, precision, **kw)
    if len(sc.fixed):
        ctx.pncg_set_dirichlet(sc.fixed, scenes.twist_targets(sc, 1))
    ctx.pncg_set_profiling(1 if profiled else 0)
    x, v = torch.tensor(x0, device=dev), torch.tensor(v0, device=dev)
    st, _ = ctx.pncg_run_dev(x, v, sc.h, frames)
    launches = ctx.pncg_get_profile()
    ctx.close()
    return x.cpu().numpy(), v.cpu().numpy(), st, launches


def _same(sc, x0, v0, frames, precision, **kw):
    xa, va, sa, _ = _run(sc, x0, v0, frames, False, precision, **kw)
    xb, vb, sb, prof = _run(sc, x0, v0, frames, True, precision, **kw)
    assert prof["grad"][1] > 0            # the other side did launch per iteration
    assert sa == sb
    assert np.array_equal(xa, xb) and np.array_equal(va, vb)
    assert np.isfinite(xa).all() and not np.array_equal(xa, x0)
    return sa


def _block(nx, ny, nz, seed=1):
    """A box on the floor, its barrier active, with a smooth velocity."""
    rng = np.random.default_rng(seed)
    sc = scenes.diff_bar_scene(seed=4, nx=nx, ny=ny, nz=nz, dx=0.01, lift=5e-4)
    v0 = 0.05 * np.sin(sc.X @ rng.uniform(5.0, 20.0, (3, 3)))
    return sc, v0


# tets: 48 (fewer than a block per XCD can share), 1,296, and the sizes around
# which the grid passes 256 and 512 logical blocks (16,384 and 32,768 tets of
# 4 lanes over 256 threads)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("dims", [(2, 2, 2), (6, 6, 6), (13, 5, 4), (14, 14, 13), (15, 14, 13), (21, 16, 16),
                                  (50, 17, 17)])
def test_bits_over_sizes(dims, precision):
    sc, v0 = _block(*dims)
    st = _same(sc, sc.X, v0, 2, precision, iter_max=20, eps=0.0, term="delta_e")
    assert all(s["iters"] == 20 for s in st)


# element terms in one to six chunks, with the records in LDS or in memory, and
# a mesh whose share fits by lane only (mixed: 2 chunks in LDS, 1, 2, 2 and 3
# in memory; float64: 2, 3, by lane or launches, 6, launches)
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("model", ["nh", "fcr"])
@pytest.mark.parametrize("dims", [(50, 17, 17), (26, 26, 27), (28, 28, 28), (150, 13, 13), (200, 12, 12)])
def test_bits_over_element_chunks(dims, model, precision):
    sc, v0 = _block(*dims)
    _same(sc, sc.X, v0, 1, precision, iter_max=6, eps=0.0, term="delta_e", model=model)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("model", ["nh", "snh", "arap", "fcr"])
def test_bits_over_materials(model, precision):
    sc, v0 = _block(17, 9, 8)
    _same(sc, sc.X, v0, 2, precision, iter_max=15, eps=0.0, term="delta_e", model=model)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("beta", ["fr", "prp", "cd", "hz"])
def test_bits_over_beta_rules(beta, precision):
    sc, v0 = _block(6, 5, 4)
    _same(sc, sc.X, v0, 1, precision, iter_max=30, eps=0.0, term="delta_e", beta=beta)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("term,eps", [("delta_e", 1e-3), ("grad_rel", 1e-2), ("grad_abs", 1e-3)])
def test_bits_over_stop_rules(term, eps, precision):
    sc, v0 = _block(9, 6, 5)
    st = _same(sc, sc.X, v0, 3, precision, iter_max=2000, eps=eps, term=term)
    # the rule, not the cap, ends every step (a step that begins within an
    # absolute tolerance makes no iteration)
    assert all(s["reason"] != 2 for s in st) and st[0]["iters"] > 0, st


def test_bits_past_one_launch():
    """1,100 iterations: two launches that reach their own limit, and a third."""
    sc, v0 = _block(6, 5, 4)
    st = _same(sc, sc.X, v0, 1, 0, iter_max=1100, eps=0.0, term="delta_e")
    assert st[0]["iters"] == 1100


@pytest.mark.parametrize("precision", [0, 1])
def test_bits_with_contact_and_rebuilds(precision):
    sc = scenes.small_contact_scene()
    v0 = np.zeros_like(sc.X)
    v0[sc.object_id == 1, 2] = -0.2
    st = _same(sc, sc.X, v0, 4, precision, iter_max=25, eps=0.0, term="delta_e")
    assert max(s["n_active"] for s in st) > 0


@pytest.mark.parametrize("precision", [0, 1])
def test_bits_of_a_falling_pile(precision):
    """A pile whose shapes meet the floor and each other: sparse contact, a
    carried list, pauses for rebuilds inside a step."""
    sc = scenes.pile_scene(n_shapes=8, target_tets=12_000)
    v0 = np.tile([0.0, 0.0, -0.3], (sc.nV, 1))
    st = _same(sc, sc.x0, v0, 12, precision, eps=1e-3, term="delta_e")
    assert sum(s["rebuilds"] for s in st) > 2 and max(s["n_active"] for s in st) > 0


def test_bits_of_the_twisted_bar():
    sc = scenes.twisted_bar_scene()
    st = _same(sc, sc.X, np.zeros_like(sc.X), 2, 1, iter_max=60, eps=0.0, term="delta_e")
    assert st[0]["rebuilds"] > 1


def test_errors_are_reported():
    """An inverted tet, and a vertex below the floor."""
    import paper_2405_08001_amd as P
    sc, v0 = _block(6, 5, 4)
    for code, move in ((P.E_INVERTED, "flip"), (P.E_PENETRATION, "sink")):
        x = sc.X.copy()
        if move == "flip":
            x[sc.tets[0, 0]] = 2 * x[sc.tets[0, 1:]].mean(0) - x[sc.tets[0, 0]]
            x[:, 2] += 0.1
        else:
            x[:, 2] -= x[:, 2].min() + 1e-4
        with pytest.raises(P.PncgError) as e:
            _run(sc, x, v0, 1, False, 0, iter_max=5, eps=0.0, term="delta_e")
        assert e.value.code == code


def test_two_contexts_on_two_threads():
    """Contexts that step at the same time on one device: each gets the bits
    it gets alone (a launch that would not fit beside the other's uses the
    per-iteration launches)."""
    import threading
    big, vbig = _block(40, 16, 16)
    small, vsmall = _block(6, 6, 6)
    jobs = [(big, vbig), (small, vsmall), (big, vbig)]
    alone = [_run(s, s.X, v, 3, False, 1, iter_max=25, eps=0.0, term="delta_e")[0] for s, v in jobs]
    got = [None] * len(jobs)

    def work(i):
        s, v = jobs[i]
        got[i] = _run(s, s.X, v, 3, False, 1, iter_max=25, eps=0.0, term="delta_e")[0]

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for a, g in zip(alone, got):
        assert np.array_equal(a, g)
