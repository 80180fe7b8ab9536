"""Acceptance words drawn in the first sweeps of a sim and ahead of the later ones: a short ka_run, one that reaches the
tenth sweep, and a short ka_sweep, against the oracle, bit for bit; one workgroup per word (2D and 3D, on
register blocks and in LDS) and tiles with one, two and three sweeps a launch, both noise modes."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noise", [0, 1])
@pytest.mark.parametrize("d,L,W", [(2, 4, 1), (2, 8, 2), (2, 16, 3), (2, 36, 1), (2, 60, 4), (2, 64, 1), (2, 68, 2), (2, 88, 3), (2, 92, 1),
                                   (2, 100, 5), (2, 132, 2), (2, 176, 1), (2, 220, 3), (2, 512, 1), (3, 4, 1), (3, 8, 2), (3, 12, 3), (3, 16, 1),
                                   (3, 16, 4), (3, 20, 2), (3, 20, 5)])
def test_calls_on_both_sides_of_the_tenth_sweep(oracle, d, L, W, noise):
    g, og = ka.ka_graph_lattice(d, L), oracle.lattice(d, L)
    R, K = 64 * W, oracle.k_from_rho(og.N, 0.65)
    sim = ka.ka_init_k(g, d, K, 9 + L, R)
    ka.ka_set_option(sim, ka.KA_OPT_NOISE, noise)
    replicas = sorted({0, R - 1})
    orc = oracle.Sim(og, d, K, 9 + L, replicas, shared=bool(noise))
    for call, n in ((ka.ka_run, 3), (ka.ka_run, 9), (ka.ka_sweep, 1)):
        call(sim, n if call is ka.ka_sweep else [orc.t + n])
        orc.sweep(n)
        words, _, f, t = ka.ka_get_state(sim)
        assert t == orc.t
        for q, b in enumerate(replicas):
            for got, bits in ((words, orc.occ), (f, orc.moved)):
                assert np.array_equal((got[b >> 6] >> np.uint64(b & 63)) & np.uint64(1), bits[q].astype(np.uint64)), (t, b)
    sim.free()
