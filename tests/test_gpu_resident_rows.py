"""Register blocks in one workgroup per word, with observations where one state exceeds the snapshot buffer (none fits)
and where one or two fit, far apart and close together, in 2D and 3D."""
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,L,W,times", [(2, 88, 34, [0, 1, 1, 2, 30]), (2, 88, 17, [0, 0, 1, 1, 1, 5]), (2, 72, 52, [2, 2, 2, 4]),
                                         (2, 64, 33, [0, 1, 3, 3, 3, 20]), (2, 64, 31, [1, 2, 2, 2, 2, 3]), (3, 20, 33, [0, 1, 1, 3]),
                                         (3, 20, 16, [0, 0, 0, 2, 2, 2, 3])])
def test_observations(oracle, d, L, W, times):
    g, og = ka.ka_graph_lattice(d, L), oracle.lattice(d, L)
    R, K = 64 * W, oracle.k_from_rho(og.N, 0.7)
    sim = ka.ka_init_k(g, d, K, 31, R)
    replicas = [0, R - 1]
    orc = oracle.Sim(og, d, K, 31, replicas)
    counts = ka.ka_run(sim, times)
    for q, t in enumerate(times):
        orc.sweep(t - orc.t)
        for row, want in zip(counts, orc.observe()):
            assert [int(row[q, b]) for b in replicas] == [int(v) for v in want], t
    sim.free()
