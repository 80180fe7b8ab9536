"""State copies in several pieces: arrays of more than 2^22 words (the staging buffer), whose pieces end
inside a word's row, on a lattice and on a graph; random words set come back as they were, and sites are
where a per-site rule puts them."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,size,R", [("lat", (3, 128), 192), ("lat", (2, 1804), 128), ("rrg", (1 << 18, 3), 1088), ("lat", (2, 180), 64),
                                         ("rrg", (32768, 4), 64), ("rrg", (32770, 4), 64)])
def test_round_trip(kind, size, R):
    g = ka.ka_graph_lattice(*size) if kind == "lat" else ka.ka_graph_rrg(size[0], size[1], 5)
    s = ka.ka_init(g, 1, 0.5, 2, R)
    W = R // 64
    rng = np.random.default_rng(7)
    arrays = [rng.integers(0, 1 << 63, size=(W, g.N), dtype=np.uint64) for _ in range(3)]
    ka.ka_set_state(s, *arrays, 9)
    n, n0, f, t = ka.ka_get_state(s)
    assert t == 9
    for x, y in zip((n, n0, f), arrays):
        assert np.array_equal(x, y)
    only = ka.ka_get_state(s, n=False, f=False)
    assert only[0] is None and only[2] is None and np.array_equal(only[1], arrays[1])
    # counts see the same words
    _, dens, ov, _ = ka.ka_observe(s)
    for b in (0, R - 1):
        bit = (arrays[0][b >> 6] >> np.uint64(b & 63)) & np.uint64(1)
        bit0 = (arrays[1][b >> 6] >> np.uint64(b & 63)) & np.uint64(1)
        assert dens[b] == int(bit.sum()) and ov[b] == int((bit & bit0).sum())
    s.free()


@pytest.mark.parametrize("N,R", [(8, 64), (10920, 64), (10922, 64), (10924, 64), (5460, 128), (5462, 128)])
def test_small_states_in_one_copy(N, R):
    """Both sides of 2^15 words in the three arrays, and one array asked for alone."""
    s = ka.ka_init(ka.ka_graph_rrg(N, 3, 5), 1, 0.5, 2, R)
    rng = np.random.default_rng(N)
    arrays = [rng.integers(0, 1 << 63, size=(R // 64, N), dtype=np.uint64) for _ in range(3)]
    ka.ka_set_state(s, *arrays, 4)
    got = ka.ka_get_state(s)
    assert got[3] == 4
    for x, y in zip(got, arrays):
        assert np.array_equal(x, y)
    only = ka.ka_get_state(s, n0=False, f=False)
    assert only[1] is None and only[2] is None and np.array_equal(only[0], arrays[0])
    s.free()
