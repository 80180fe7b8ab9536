"""Lattice passes that load the moved-ever words with the state words (few edge-words a launch) and
those that load them late give the same state: replicas do not depend on how many others are
simulated, so 64 replicas of a launch on one side of the line equal the first 64 of more replicas on
the other side, in 2D and 3D, for one and two words per thread."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,L,R,m", [(3, 128, 128, 3), (3, 100, 256, 3), (3, 128, 192, 5), (2, 1024, 192, 2)])
def test_both_sides_of_the_line(d, L, R, m):
    # edges of a class x words: N/4 x 1 is at most 2^19, N/4 x R/64 is above it
    g = ka.ka_graph_lattice(d, L)
    assert L ** d // 4 <= 1 << 19 < L ** d // 4 * (R // 64)
    states = []
    for r in (64, R):
        sim = ka.ka_init(g, m, 0.8, 5, r)
        ka.ka_set_option(sim, ka.KA_OPT_PATH, 1)
        ka.ka_sweep(sim, 3)
        states.append(ka.ka_get_state(sim))
        sim.free()
    for a, b in zip(states[0][:3], states[1][:3]):
        assert np.array_equal(a[0], b[0])
    assert np.any(states[0][2])
