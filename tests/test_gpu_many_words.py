"""Replica counts whose words, or whose replicas times 1024 threads, exceed one grid (2^16 workgroups in y,
2^32 threads in x): the initial state, a few sweeps and the counts, on both sides of the selection's
size limit."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [65534, 65600, 65537, 131074])
def test_every_replica_is_initialised(oracle, W):
    g, og = ka.ka_graph_lattice(2, 4), oracle.lattice(2, 4)
    K, R = 7, 64 * W
    sim = ka.ka_init_k(g, 2, K, 3, R)
    _, dens, ov, pers = ka.ka_observe(sim)
    assert (dens == K).all() and (ov == K).all() and (pers == K).all()
    replicas = sorted({0, 63, 4096, 64 * (W - 65536) + 1 if W > 65536 else 1, R // 2, R - 65, R - 1})
    orc = oracle.Sim(og, 2, K, 3, replicas)
    dens, ov, pers = ka.ka_run(sim, [1, 3])
    n, n0, f, _ = ka.ka_get_state(sim)
    orc.sweep(3)
    counts = orc.observe()
    for q, b in enumerate(replicas):
        for words, bits in ((n, orc.occ), (n0, orc.occ0), (f, orc.moved)):
            assert np.array_equal((words[b >> 6] >> np.uint64(b & 63)) & np.uint64(1), bits[q].astype(np.uint64)), b
        assert (dens[1, b], ov[1, b], pers[1, b]) == tuple(c[q] for c in counts)
    sim.free()


def test_every_replica_is_initialised_by_the_window_selection(oracle):
    g, K, R = ka.ka_graph_lattice(2, 128), 5000, 64 * 65600
    sim = ka.ka_init_k(g, 2, K, 3, R)   # 26 GB
    _, dens, ov, pers = ka.ka_observe(sim)
    assert (dens == K).all() and (ov == K).all() and (pers == K).all()
    sim.free()
