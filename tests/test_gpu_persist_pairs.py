"""The pair terms of the persistent iteration kernel against those of the
per-iteration launches (which a context uses while its profiling is on), over
the frames in which the shapes of a pile come to touch.  A product or sum
fused in another order shows in the last place of the curvature of a few
pairs, and in a step's bits only now and then, so the run is long, in float64
and mixed, for each material, with the projected and the full barrier
Hessian."""
import numpy as np
import pytest

import scenes
from helpers import make_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,model,full,frames", [
    (0, "nh", False, 60), (0, "nh", True, 40), (0, "snh", False, 60), (0, "fcr", False, 60),
    (1, "nh", False, 60), (1, "snh", False, 60), (1, "arap", False, 60), (1, "fcr", False, 60)])
def test_bits_while_shapes_come_to_touch(precision, model, full, frames):
    import torch
    sc = scenes.pile_scene()
    dev = torch.device("cuda:0")
    out = []
    for profiled in (0, 1):
        ctx = make_ctx(sc, precision, model=model, barrier_full=full)
        ctx.pncg_set_profiling(profiled)
        x, v = torch.tensor(sc.x0, device=dev), torch.tensor(sc.v0, device=dev)
        st, _ = ctx.pncg_run_dev(x, v, sc.h, frames)
        ctx.close()
        out.append((x.cpu().numpy(), v.cpu().numpy(), st))
    (xa, va, sa), (xb, vb, sb) = out
    assert max(s["n_active"] for s in sa) >= 10
    assert sa == sb
    assert np.array_equal(xa, xb) and np.array_equal(va, vb)
