"""Argument checks of the persistent kernels' settings (no GPU needed)."""
import pytest


def test_wait_limit_is_checked():
    import paper_2405_08001_amd as P
    c = P.Context(0, P.FP64)
    for us in (0, 1, 20000, -1):
        c.pncg_set_persistent(us)
    with pytest.raises(P.PncgError) as e:
        c.pncg_set_persistent(-2)
    assert e.value.code == P.E_INVAL
    assert c.pncg_get_persistent() == (0, 0)
    c.close()
