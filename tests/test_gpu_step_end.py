"""The end of a step on the per-iteration launches that stops by its rule in
the chunk of launches before the last: when the call returns its outputs are
complete, for a reader on any stream, and what the output kernel finds wrong
with them is reported.  (The stop rule holds at the first iteration, in the
chunk [0, 16); [16, 32), which ends with the output kernel, is sent ahead.)"""
import dataclasses

import numpy as np
import pytest

import scenes
from helpers import make_ctx

pytestmark = pytest.mark.gpu

STOP = dict(iter_max=31, eps=2.0, term="delta_e", chunk=16)


def _scene(kind):
    """(scene, precision, context options, steps that lead to the launches)"""
    if kind == "large":          # a block's share does not fit in LDS
        return scenes.diff_bar_scene(seed=4, nx=200, ny=12, nz=12, dx=0.01, lift=5e-4), 0, {}, 0
    if kind == "dense":          # known to be dense after the first step
        return scenes.packed_pile_scene(n_shapes=9, target_tets=21_000), 1, {}, 1
    return scenes.small_contact_scene(), 0, dict(split=True) if kind == "split" else dict(scatter=1), 0


# (the split step is not allocation-free)
@pytest.mark.parametrize("kind,call", [(k, c) for k in ("large", "dense", "split", "atomic")
                                       for c in ("step_dev", "step_dev_noalloc", "run_dev")
                                       if (k, c) != ("split", "step_dev_noalloc")])
def test_outputs_are_complete_on_return(kind, call):
    import torch
    sc, precision, kw, lead = _scene(kind)
    dev = torch.device("cuda:0")
    ctx = make_ctx(sc, precision, **kw, **STOP)
    if sc.self_contact:
        ctx.pncg_set_tuning(skin=40.0 * sc.dhat)     # a chunk is not cut short for the list
    x, v = torch.tensor(sc.x0, device=dev), torch.tensor(sc.v0, device=dev)
    xo, vo = torch.empty_like(x), torch.empty_like(v)
    for _ in range(lead):
        st = ctx.pncg_step_dev(x, v, sc.h, xo, vo)
        assert 4 * st["n_candidates"] > sc.nV
    if call == "step_dev_noalloc" and sc.self_contact:
        ctx.pncg_step_dev(x, v, sc.h, xo, vo)        # sizes the contact buffers
    for _ in range(3):
        if call == "run_dev":
            xo.copy_(x)
            vo.copy_(v)
            torch.cuda.synchronize()
            st = ctx.pncg_run_dev(xo, vo, sc.h, 1)[0][0]
        else:
            xo.fill_(float("nan"))
            vo.fill_(float("nan"))
            torch.cuda.synchronize()
            st = getattr(ctx, "pncg_" + call)(x, v, sc.h, xo, vo)
        xa, va = xo.clone(), vo.clone()              # on torch's stream, right behind the call
        torch.cuda.synchronize()
        assert st["iters"] == 1 and st["reason"] == 0
        assert torch.equal(xa, xo) and torch.equal(va, vo)
        assert torch.isfinite(xa).all() and not torch.equal(xa, x)
    # the host-pointer step, whose copies follow on the context's own stream
    xh, vh, sh = ctx.pncg_step(sc.x0, sc.v0, sc.h)
    assert sh["iters"] == 1
    xa, va = xa.cpu().numpy(), va.cpu().numpy()
    if kind == "atomic":         # sums in the order the atomics come: a few roundings of terms up to 1e3 times the sum
        assert np.allclose(xa, xh, rtol=0.0, atol=1e-11 * np.abs(sc.X).max())
    else:
        assert np.array_equal(xa, xh) and np.array_equal(va, vh)
    ctx.close()


@pytest.mark.parametrize("host", [False, True])
def test_non_finite_result_is_reported(host):
    """A vertex without tets, an object of its own: its diagonal is zero, so
    its direction is not a number, while the other object's iteration stops by
    the rule.  Only the output kernel sees it."""
    import torch
    import paper_2405_08001_amd as P
    sc = scenes.diff_bar_scene(seed=4, nx=6, ny=5, nz=4, dx=0.01, lift=0.01)
    sc = dataclasses.replace(sc, X=np.vstack([sc.X, [[1.0, 1.0, 1.0]]]), x0=np.vstack([sc.x0, [[1.0, 1.0, 1.0]]]),
                             v0=np.vstack([sc.v0, np.zeros((1, 3))]),
                             object_id=np.append(np.zeros(sc.nV, np.int32), np.int32(1)), planes=np.zeros((0, 4)))
    ctx = make_ctx(sc, 0, split=True, **STOP)
    dev = torch.device("cuda:0")
    x, v = torch.tensor(sc.x0, device=dev), torch.tensor(sc.v0, device=dev)
    with pytest.raises(P.PncgError) as e:
        if host:
            ctx.pncg_step(sc.x0, sc.v0, sc.h)
        else:
            ctx.pncg_step_dev(x, v, sc.h, torch.empty_like(x), torch.empty_like(v))
    assert e.value.code == P.E_NONFINITE
    ctx.close()
