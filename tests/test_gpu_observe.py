"""Per-replica counts against a plain numpy count of the exported state, bit for bit, at the edges
of the observation kernel's work split: one partial wave, remainders of the four sites a lane takes
at a time, several workgroups per plane, and lanes that empty their counters several times."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


def numpy_counts(words, replicas):
    """Number of set bits of each listed replica in words [W][N]."""
    out = []
    for b in replicas:
        out.append(int(((words[b >> 6] >> np.uint64(b & 63)) & np.uint64(1)).sum()))
    return np.array(out)


@pytest.mark.parametrize("d,L,R", [(2, 4, 64), (2, 4, 128), (2, 8, 192), (3, 4, 320), (2, 24, 64), (2, 44, 128), (2, 68, 64),
                                   (2, 180, 128), (3, 60, 192), (3, 100, 128), (3, 256, 64)])
def test_counts_equal_numpy(d, L, R):
    g = ka.ka_graph_lattice(d, L)
    s = ka.ka_init(g, 2 * d - 2, 0.6, 11, R)
    ka.ka_sweep(s, 2)
    replicas = range(R) if g.N < 1 << 19 else [0, 1, 31, 32, 47, 63, R - 1]
    dens, ov, pers = ka.ka_run(s, [2, 2, 3])   # two rows of one state, then the next one's
    for row in range(2):
        assert np.array_equal(dens[row], dens[0]) and np.array_equal(ov[row], ov[0]) and np.array_equal(pers[row], pers[0])
    n, n0, f, t = ka.ka_get_state(s)
    assert t == 3 and (dens == s.K).all()
    sel = list(replicas)
    assert np.array_equal(dens[2][sel], numpy_counts(n, sel))
    assert np.array_equal(ov[2][sel], numpy_counts(n & n0, sel))
    assert np.array_equal(pers[2][sel], numpy_counts(n0 & ~f, sel))
    s.free()
