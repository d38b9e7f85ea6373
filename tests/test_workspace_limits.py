"""Workspace sizes that callers hold: what was enough stays enough."""
import pytest


@pytest.fixture(scope="module")
def mpr():
    import paper_2409_17658_amd as m

    m.lib()
    return m


def _up(x, a=256):
    return (x + a - 1) // a * a


@pytest.mark.parametrize("n", [1, 5, 31, 32, 33, 97, 200, 256, 257, 287, 848, 21909])
def test_period_workspace_is_the_ring_and_8n_bytes(mpr, n):
    """The ring of powers and, before it, 8 n bytes and one line of scalars."""
    slot = _up(2 * n * _up(n, 8)) + _up(8 * n)
    for slots in (2, 9):
        assert mpr.period_workspace_size(n, slots) == _up(_up(8 * n) + 64) + slots * slot
