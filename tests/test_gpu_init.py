"""Initial states against the oracle's, bit for bit, around the smallest size of the window
selection (2^14 sites) and at particle numbers where the window meets 0 or N; and two seeds
whose threshold lies outside the window (found with a plain CPU count of the keys), so that the
replica is selected over all its keys."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


def check(oracle, lib_graph, or_graph, K, seed, R, replicas):
    sim = ka.ka_init_k(lib_graph, 1, K, seed, R)
    n, n0, f, _ = ka.ka_get_state(sim)
    _, dens, ov, pers = ka.ka_observe(sim)
    sim.free()
    assert (dens == K).all() and (ov == K).all() and (pers == K).all()
    assert np.array_equal(n, n0) and not f.any()
    orc = oracle.Sim(or_graph, 1, K, seed, replicas)
    for q, b in enumerate(replicas):
        bits = (n[b >> 6] >> np.uint64(b & 63)) & np.uint64(1)
        assert np.array_equal(bits.astype(np.uint8), orc.occ0[q].astype(np.uint8)), (K, seed, b)


@pytest.mark.parametrize("d,L,R", [(2, 124, 64), (2, 128, 64), (2, 128, 192), (2, 132, 128), (3, 28, 256)])
def test_lattice_initial_state(oracle, d, L, R):
    g, og = ka.ka_graph_lattice(d, L), oracle.lattice(d, L)
    N = L ** d
    for K in (0, 1, 13, N // 2, int(0.85 * N), N - 13, N - 1, N):
        check(oracle, g, og, K, 5 + K, R, sorted({0, 1, 31, 32, 63, R // 2, R - 1}))


@pytest.mark.parametrize("N,z,R", [(16382, 3, 64), (16384, 5, 128), (50000, 4, 64)])
def test_graph_initial_state(oracle, N, z, R):
    g, og = ka.ka_graph_rrg(N, z, 3), oracle.rrg(N, z, 3)
    for K in (1, N // 3, int(0.7 * N), N - 1):
        check(oracle, g, og, K, 9 + K, R, sorted({0, 33, R - 1}))


@pytest.mark.parametrize("seed,replica", [(7088, 34), (9339, 57), (20746, 37)])
def test_threshold_outside_the_window(oracle, seed, replica):
    check(oracle, ka.ka_graph_lattice(2, 128), oracle.lattice(2, 128), 8192, seed, 64, [replica - 1, replica, replica + 1])
