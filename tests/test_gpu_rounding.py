"""The persistent kernels and a launch per iteration round every term alike.
In a mesh of one tet no sum hides a term's last place, so a product fused in
another order shows in the predicted decrease or the gradient's norm of some
of the states: deformed and moving, in and out of a plane's barrier."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model", ["nh", "snh", "arap", "fcr"])
@pytest.mark.parametrize("precision", [0, 1])
def test_one_tet(precision, model):
    import paper_2405_08001_amd as P
    tri = np.array([[1, 2, 3], [0, 3, 2], [0, 1, 3], [0, 2, 1]])
    edge = np.array([[0, 1], [0, 2], [0, 3], [1, 2], [1, 3], [2, 3]])
    adjoints = 0
    for seed in range(40):
        rng = np.random.default_rng(seed)
        X = 0.1 * np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [0, 0, 1.0]]) + rng.uniform(-0.01, 0.01, (4, 3))
        x, v = X + rng.uniform(-0.008, 0.008, (4, 3)), rng.uniform(-0.5, 0.5, (4, 3))
        n = np.array([0.1 * seed / 40, 0.2, 1.0])
        n /= np.linalg.norm(n)
        plane = np.array([[*n, (x @ n).min() - 4e-4]])
        out = []
        for profiled in (0, 1):
            c = P.Context(0, precision)
            c.pncg_set_model(model)
            c.pncg_set_mesh(X, np.array([[0, 1, 2, 3]]), tri, edge)
            c.pncg_set_material(np.array([1e5 * (1 + seed / 7)]), 0.3 + 0.004 * seed, 1000.0)
            c.pncg_set_contact(1e-3, 1e4, 0.0, plane if seed % 2 else None, 0)
            c.pncg_set_solver(3, 0.0, P.TERM_DELTA_E, (0.0, 0.0, -9.8), 0)
            c.pncg_set_profiling(profiled)
            r = list(c.pncg_step(x, v, 1 / 60))
            assert c.pncg_get_persistent()[0] == 1 - profiled
            if precision == 0:
                try:
                    r += c.pncg_adjoint_step(x, 1 / 60, v, x, cg_tol=0.0, cg_max=4)
                    adjoints += 1
                except P.PncgError as e:       # an indefinite H, on both sides
                    assert e.code == P.E_INDEFINITE
            c.close()
            out.append(r)
        assert len(out[0]) == len(out[1]), seed
        for a, b in zip(*out):
            assert a == b if isinstance(a, dict) else np.array_equal(a, b), seed
    assert precision == 1 or adjoints > 40
