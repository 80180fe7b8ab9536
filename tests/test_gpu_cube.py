"""Small 3D lattices on register blocks (one workgroup per word) against the oracle, bit for bit: both
sizes of the workgroup, blocks that do not fill a wave, lattices of one block per plane, odd and
even word counts, both noise modes, chunks and snapshots in ka_run, and, in 2D and 3D, so many words that
they are drawn in the sweep; and the smallest 3D lattices (L = 4 to 12), which keep n and f in LDS."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


def unpack(words, b):
    return ((words[b >> 6] >> np.uint64(b & 63)) & np.uint64(1)).astype(np.uint8)


def check_state(sim, orc, replicas):
    n, n0, f, t = ka.ka_get_state(sim)
    assert t == orc.t
    for q, b in enumerate(replicas):
        assert np.array_equal(unpack(n, b), orc.occ[q].astype(np.uint8)), b
        assert np.array_equal(unpack(f, b), orc.moved[q].astype(np.uint8)), b


@pytest.mark.parametrize("noise", [0, 1])
@pytest.mark.parametrize("L,R,m", [(4, 64, 5), (4, 192, 3), (8, 128, 3), (12, 64, 4), (12, 320, 2), (16, 64, 3), (16, 256, 3), (20, 64, 3),
                                   (20, 128, 5), (20, 192, 3), (20, 256, 4)])
def test_one_workgroup(oracle, L, R, m, noise):
    g, og = ka.ka_graph_lattice(3, L), oracle.lattice(3, L)
    K = oracle.k_from_rho(og.N, 0.7)
    sim = ka.ka_init_k(g, m, K, 7 + L, R)
    ka.ka_set_option(sim, ka.KA_OPT_NOISE, noise)
    replicas = sorted({0, 63, R // 2, R - 1})
    orc = oracle.Sim(og, m, K, 7 + L, replicas, shared=bool(noise))
    for n in (1, 2, 5):
        ka.ka_sweep(sim, n)
        orc.sweep(n)
    check_state(sim, orc, replicas)
    sim.free()


@pytest.mark.parametrize("L,R,times", [(8, 64, [0, 1, 1, 2, 7, 7]), (20, 64, list(range(0, 60, 2))), (20, 256, [0, 1, 5, 5, 5, 11, 24]),
                                       (20, 2816, [0, 2, 2, 3])])
def test_observation_times(oracle, L, R, times):
    g, og = ka.ka_graph_lattice(3, L), oracle.lattice(3, L)
    K = oracle.k_from_rho(og.N, 0.75)
    sim = ka.ka_init_k(g, 3, K, 31, R)
    replicas = [0, R - 1]
    orc = oracle.Sim(og, 3, K, 31, replicas)
    dens, ov, pers = ka.ka_run(sim, times)
    for q, t in enumerate(times):
        orc.sweep(t - orc.t)
        od, oo, op = orc.observe()
        for k, b in enumerate(replicas):
            assert (dens[q, b], ov[q, b], pers[q, b]) == (od[k], oo[k], op[k]), (t, b)
    check_state(sim, orc, replicas)
    sim.free()


@pytest.mark.parametrize("d,L,W", [(3, 4, 1367), (3, 12, 220), (3, 16, 87), (3, 20, 181), (2, 8, 8193), (2, 64, 130), (2, 88, 72)])
def test_words_drawn_in_the_sweep(oracle, d, L, W):
    g, og = ka.ka_graph_lattice(d, L), oracle.lattice(d, L)
    R = 64 * W
    K = oracle.k_from_rho(og.N, 0.7)
    sim = ka.ka_init_k(g, d, K, 5, R)
    replicas = [0, 64 * (W // 2) + 1, R - 65, R - 1]
    orc = oracle.Sim(og, d, K, 5, replicas)
    ka.ka_sweep(sim, 3)
    orc.sweep(3)
    check_state(sim, orc, replicas)
    sim.free()
