"""State copies on both sides of the size up to which the three arrays travel in one copy (7 * 2^13 words), on a
graph and on a lattice, whole and one array alone."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,size,R", [("rrg", (19114, 3), 64), ("rrg", (19116, 3), 64), ("rrg", (100, 3), 8192), ("lat", (2, 136), 64),
                                         ("lat", (2, 140), 64), ("lat", (2, 16), 4736), ("lat", (2, 16), 4800)])
def test_round_trip(kind, size, R):
    g = ka.ka_graph_lattice(*size) if kind == "lat" else ka.ka_graph_rrg(*size, 5)
    s = ka.ka_init(g, 1, 0.5, 2, R)
    rng = np.random.default_rng(g.N)
    arrays = [rng.integers(0, 1 << 63, size=(R // 64, g.N), dtype=np.uint64) for _ in range(3)]
    ka.ka_set_state(s, *arrays, 4)
    got = ka.ka_get_state(s)
    assert got[3] == 4
    for x, y in zip(got, arrays):
        assert np.array_equal(x, y)
    only = ka.ka_get_state(s, n=False, n0=False)
    assert only[0] is None and only[1] is None and np.array_equal(only[2], arrays[2])
    s.free()
