"""A ka_sweep captured into a HIP graph, with direct sweeps and a restored state between the replays: each
replay runs the captured sweeps on the sim's state as it then is.  One size for each way a
sweep can run: 2D in one workgroup and in tiles, 3D and graphs."""
import numpy as np
import pytest
import torch

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,size,R", [("lat", (2, 32), 64), ("lat", (2, 92), 128), ("lat", (2, 128), 64), ("lat", (2, 256), 192),
                                         ("lat", (3, 24), 64), ("rrg", (20000, 4), 64)])
def test_replays_between_direct_sweeps(oracle, kind, size, R):
    if kind == "lat":
        g, og = ka.ka_graph_lattice(*size), oracle.lattice(*size)
    else:
        g, og = ka.ka_graph_rrg(*size, 3), oracle.rrg(*size, 3)
    K = oracle.k_from_rho(og.N, 0.6)
    stream = torch.cuda.Stream()
    sim = ka.ka_init_k(g, 2, K, 5, R, stream=stream)
    replicas = [0, R - 1]
    ka.ka_sweep(sim, 1)
    start = ka.ka_get_state(sim)

    def check(sweeps):
        orc = oracle.Sim(og, 2, K, 5, replicas)
        orc.sweep(sweeps)
        n, _, f, _ = ka.ka_get_state(sim)
        for q, b in enumerate(replicas):
            for words, bits in ((n, orc.occ), (f, orc.moved)):
                assert np.array_equal((words[b >> 6] >> np.uint64(b & 63)) & np.uint64(1), bits[q].astype(np.uint64)), (sweeps, b)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        graph.capture_begin(capture_error_mode="thread_local")
        ka.ka_sweep(sim, 2)      # sweeps 1 and 2
        graph.capture_end()
    check(1)
    for direct in (1, 2, 4):     # an odd number of launches on tiles, and an even one
        with torch.cuda.stream(stream):
            graph.replay()
        check(3)
        ka.ka_set_state(sim, *start[:3], 3)
        ka.ka_sweep(sim, direct)
        ka.ka_set_state(sim, *start)
    with torch.cuda.stream(stream):
        graph.replay()
    check(3)
    sim.free()
