"""Lattices with so many words that their planes run in LDS, a thread per edge or three (both sides of the lines to the
register blocks and tiles, odd and even word counts, both noise modes, words drawn ahead and in the loop), or as
class passes instead of tiles; and observations of more rows than the snapshots hold, of one row and of
none, counted after the launches or in the loop.  Against the oracle, bit for bit."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


def check_state(sim, orc, replicas):
    n, _, f, t = ka.ka_get_state(sim)
    assert t == orc.t
    for q, b in enumerate(replicas):
        for words, bits in ((n, orc.occ), (f, orc.moved)):
            assert np.array_equal((words[b >> 6] >> np.uint64(b & 63)) & np.uint64(1), bits[q].astype(np.uint64)), b


@pytest.mark.parametrize("noise", [0, 1])
@pytest.mark.parametrize("d,L,W", [(2, 12, 333), (2, 12, 334), (2, 16, 251), (2, 24, 166), (2, 24, 167), (2, 32, 256), (2, 40, 99), (2, 40, 100),
                                   (2, 44, 256), (2, 44, 257), (2, 48, 258), (2, 52, 258), (2, 92, 59), (2, 92, 61), (2, 96, 65), (2, 92, 160), (2, 100, 162), (3, 4, 65), (3, 8, 68), (3, 8, 69), (3, 12, 20),
                                   (3, 12, 21), (3, 16, 27), (3, 16, 29), (3, 16, 256), (3, 16, 257), (3, 16, 258)])
def test_sweeps(oracle, d, L, W, noise):
    g, og = ka.ka_graph_lattice(d, L), oracle.lattice(d, L)
    R, m, K = 64 * W, d, oracle.k_from_rho(og.N, 0.65)
    sim = ka.ka_init_k(g, m, K, 7 + L, R)
    ka.ka_set_option(sim, ka.KA_OPT_NOISE, noise)
    replicas = sorted({0, 63, 64 * (W // 2) + 5, R - 64, R - 1})
    orc = oracle.Sim(og, m, K, 7 + L, replicas, shared=bool(noise))
    for n in (1, 3):
        ka.ka_sweep(sim, n)
        orc.sweep(n)
    check_state(sim, orc, replicas)
    sim.free()


# snapshot rows of 4 MiB: L = 8 x 2048 replicas 16, x 16384 2; L = 40 x 8192 1; L = 48 x 16448 none
@pytest.mark.parametrize("d,L,W,times", [(3, 8, 32, [0, 0] + list(range(1, 40)) + [40] * 20 + [41]), (3, 8, 256, [1, 1, 1, 2, 5, 5, 9]),
                                         (3, 4, 2, list(range(0, 90, 3))), (2, 24, 256, [0, 1, 1, 4, 4, 4, 6]), (2, 40, 128, [0, 0, 2, 3, 3, 7]),
                                         (2, 48, 257, [0, 1, 1, 4]), (3, 12, 7, [3] * 30 + [4]),
                                         (2, 48, 193, [0, 1, 1, 2, 4]), (2, 64, 40, [1, 2, 2, 3, 6]), (2, 64, 40, [0, 0, 0, 0, 60]),
                                         (3, 16, 33, [0, 1, 2, 3]), (3, 16, 8, list(range(12))), (2, 92, 61, [0, 0, 2])])
def test_observations(oracle, d, L, W, times):
    g, og = ka.ka_graph_lattice(d, L), oracle.lattice(d, L)
    R, m, K = 64 * W, d, oracle.k_from_rho(og.N, 0.7)
    sim = ka.ka_init_k(g, m, K, 31, R)
    replicas = [0, R - 1]
    orc = oracle.Sim(og, m, K, 31, replicas)
    dens, ov, pers = ka.ka_run(sim, times)
    for q, t in enumerate(times):
        orc.sweep(t - orc.t)
        for row, want in zip((dens, ov, pers), orc.observe()):
            assert [int(row[q, b]) for b in replicas] == [int(v) for v in want], t
    check_state(sim, orc, replicas)
    sim.free()
