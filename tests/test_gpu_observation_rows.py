"""Observation times of one-workgroup sweeps: as many as travel with a launch, one fewer, one more
and far more, some of them equal, in 2D and 3D, against counts taken between class passes."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,L,R,m", [(2, 32, 64, 2), (2, 64, 192, 2), (3, 16, 64, 3), (3, 20, 128, 3)])
@pytest.mark.parametrize("rows", [1, 15, 16, 17, 40])
def test_rows(d, L, R, m, rows):
    g = ka.ka_graph_lattice(d, L)
    first = 3
    times = [first + (2 * q) // 3 for q in range(rows)]
    counts = []
    for path in (0, 1):
        sim = ka.ka_init(g, m, 0.7, 11, R)
        ka.ka_set_option(sim, ka.KA_OPT_PATH, path)
        ka.ka_sweep(sim, 2)
        counts.append(ka.ka_run(sim, times))
        sim.free()
    for a, b in zip(*counts):
        assert np.array_equal(np.asarray(a), np.asarray(b))
