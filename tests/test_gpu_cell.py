"""Candidate lists over the grid's cell sizes: a caller's cell that is finer
than the size derived from the surface is grouped, 2^shift cells to a side, and
neither the lists nor which states fit may depend on that."""
import numpy as np
import pytest

import scenes
from helpers import check_solver_pairs, make_ctx, make_problem

pytestmark = pytest.mark.gpu


# 0 the derived cell; the others in units of it: coarser, ungrouped, the first
# that is grouped in twos, in fours, in sixteens
@pytest.mark.parametrize("unit", [0.0, 3.0, 0.75, 0.66, 0.3, 0.06])
@pytest.mark.parametrize("offset", [0.0, -0.35])
def test_lists_do_not_depend_on_the_cell(unit, offset):
    import paper_2405_08001_amd as L
    sc = scenes.small_contact_scene()
    prob = make_problem(sc)
    skin = 2.0 * sc.dhat
    e = sc.X[sc.edges]
    derived = max(1.5 * float(np.mean(np.linalg.norm(e[:, 0] - e[:, 1], axis=1))), sc.dhat + skin)
    ctx = make_ctx(sc, 0, cell=unit * derived)
    ctx.pncg_set_tuning(skin=skin)
    x = sc.X + offset            # cells of either sign
    pt, ee, _ = prob.candidate_lists(x)
    assert len(pt) > 0 and len(ee) > 0
    assert np.array_equal(ctx.pncg_candidates(x, L.KIND_PT), pt)
    assert np.array_equal(ctx.pncg_candidates(x, L.KIND_EE), ee)
    n_pt, n_ee = check_solver_pairs(ctx, prob, x, sc.dhat + skin)
    print(f"cell {unit} offset {offset}: PT {n_pt} EE {n_ee}", flush=True)
    assert n_pt > 0 and n_ee > 0
