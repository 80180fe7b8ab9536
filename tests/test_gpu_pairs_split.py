"""Four-point sums where the displacements of a tile are split over workgroups, in few and in many parts
(lists that the parts do not divide), and where gathers take the tiles' place although they would fit."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka
from test_gpu_pairs import sums

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,L,R,r2_max", [(2, 8, 320, 13), (2, 16, 64, 100), (2, 40, 64, 400), (2, 40, 1024, 400), (2, 96, 320, 100), (2, 128, 192, 61),
                                          (2, 512, 128, 4), (3, 4, 64, 3), (3, 12, 1024, 100), (3, 16, 320, 41), (3, 24, 64, 400), (3, 32, 128, 1)])
def test_pair_sums_equal_autocorrelations(d, L, R, r2_max):
    s = ka.ka_init(ka.ka_graph_lattice(d, L), 2 * d - 2, 0.6, 23, R)
    ka.ka_sweep(s, 2)
    S2, S11, cnt = ka.ka_observe_pairs(s, r2_max)
    n, n0, _, _ = ka.ka_get_state(s)
    s.free()
    eS2, eS11, ecnt = sums(n, n0, d, L, R, r2_max)
    assert np.array_equal(cnt, ecnt)
    assert np.array_equal(S2, eS2)
    assert np.array_equal(S11, eS11)
