"""2D lattices on register blocks against the oracle, bit for bit: one workgroup per word up to
L = 128 (every size of its workgroup, blocks that do not fill the last wave, lattices of one block),
tiles above it (ragged last tiles, tiles that wrap, acceptance words drawn ahead or in the sweep),
both noise modes, odd and even word counts, and the arrangement of chunks and snapshots in ka_run."""
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
@pytest.mark.parametrize("L,R,m", [(4, 64, 3), (8, 128, 2), (16, 64, 1), (32, 64, 2), (36, 192, 2), (60, 64, 2), (64, 256, 2), (68, 64, 3),
                                   (88, 128, 2), (92, 64, 2), (100, 320, 2), (128, 64, 2), (128, 128, 1)])
def test_one_workgroup(oracle, L, R, m, noise):
    g, og = ka.ka_graph_lattice(2, L), oracle.lattice(2, L)
    K = oracle.k_from_rho(og.N, 0.65)
    sim = ka.ka_init_k(g, m, K, 7 + L, R)
    ka.ka_set_option(sim, ka.KA_OPT_NOISE, noise)
    replicas = sorted({0, 63, R // 2, R - 1})
    orc = oracle.Sim(og, m, K, 7 + L, replicas, shared=bool(noise))
    for n in (1, 2, 4):
        ka.ka_sweep(sim, n)
        orc.sweep(n)
    check_state(sim, orc, replicas)
    sim.free()


@pytest.mark.parametrize("L,R,noise", [(132, 64, 0), (132, 192, 1), (140, 128, 0), (176, 64, 0), (180, 64, 0), (220, 320, 0), (512, 128, 0),
                                       (512, 192, 0), (724, 128, 0), (728, 64, 1), (1028, 64, 0)])
def test_tiles(oracle, L, R, noise):
    g, og = ka.ka_graph_lattice(2, L), oracle.lattice(2, L)
    K = oracle.k_from_rho(og.N, 0.7)
    sim = ka.ka_init_k(g, 2, K, 3 + L, R)
    ka.ka_set_option(sim, ka.KA_OPT_NOISE, noise)
    replicas = sorted({0, R - 1})
    orc = oracle.Sim(og, 2, K, 3 + L, replicas, shared=bool(noise))
    ka.ka_sweep(sim, 1)
    ka.ka_run(sim, [2, 4])
    orc.sweep(4)
    check_state(sim, orc, replicas)
    # the class passes give the same whole state
    other = ka.ka_init_k(g, 2, K, 3 + L, R)
    ka.ka_set_option(other, ka.KA_OPT_NOISE, noise)
    ka.ka_set_option(other, ka.KA_OPT_PATH, 1)
    ka.ka_sweep(other, 4)
    for x, y in zip(ka.ka_get_state(sim), ka.ka_get_state(other)):
        assert np.array_equal(np.asarray(x), np.asarray(y))
    sim.free()
    other.free()


def test_many_sweeps_and_a_restored_state(oracle):
    """Chunks of words drawn ahead on the tiles (8 sweeps at L = 256 with 4 words), an odd number
    of swaps between exports, and a state set back."""
    L, R = 256, 256
    g, og = ka.ka_graph_lattice(2, L), oracle.lattice(2, L)
    K = oracle.k_from_rho(og.N, 0.7)
    sim = ka.ka_init_k(g, 2, K, 19, R)
    orc = oracle.Sim(og, 2, K, 19, [0, 255])
    ka.ka_sweep(sim, 11)
    saved = ka.ka_get_state(sim)
    ka.ka_sweep(sim, 6)
    first = ka.ka_get_state(sim)
    ka.ka_set_state(sim, *saved)
    ka.ka_sweep(sim, 5)
    ka.ka_sweep(sim, 1)
    again = ka.ka_get_state(sim)
    for x, y in zip(first, again):
        assert np.array_equal(np.asarray(x), np.asarray(y))
    orc.sweep(17)
    check_state(sim, orc, [0, 255])
    sim.free()


@pytest.mark.parametrize("L,R,times", [
    (64, 64, [0, 0, 1, 1, 5, 5, 5, 6, 40]),
    (64, 64, [3] * 70 + [4] * 3 + [9]),          # more rows at one time than the snapshots hold
    (64, 64, list(range(0, 150))),
    (128, 256, [0, 1, 2, 3, 3, 3, 3, 3, 4, 5, 5, 20, 33, 33]),
    (128, 1088, [0, 1, 1, 2]),                   # one state exceeds the snapshot buffer
])
def test_observation_times(oracle, L, R, times):
    g, og = ka.ka_graph_lattice(2, L), oracle.lattice(2, L)
    K = oracle.k_from_rho(og.N, 0.7)
    sim = ka.ka_init_k(g, 2, K, 31, R)
    replicas = [0, R - 1]
    orc = oracle.Sim(og, 2, K, 31, replicas)
    dens, ov, pers = ka.ka_run(sim, times)
    for q, t in enumerate(times):
        orc.sweep(t - orc.t)
        od, oo, op = orc.observe()
        for k, b in enumerate(replicas):
            assert (dens[q, b], ov[q, b], pers[q, b]) == (od[k], oo[k], op[k]), (t, b)
    check_state(sim, orc, replicas)
    sim.free()
