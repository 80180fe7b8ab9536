"""Device memory that calls take: counting the state as it is takes no buffer that only sweeps need."""
import pytest
import torch

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info(0)[0]


# What a sweep would allocate: a second copy of n (32 MiB), or words drawn ahead and snapshots (12 MiB)
@pytest.mark.parametrize("kind,size,R", [("lat", (2, 1024), 256), ("lat", (2, 64), 64), ("lat", (3, 20), 64), ("lat", (3, 8), 64),
                                         ("rrg", (2000, 4), 64)])
def test_observation_takes_no_sweep_buffers(kind, size, R):
    g = ka.ka_graph_lattice(*size) if kind == "lat" else ka.ka_graph_rrg(*size, 5)
    s = ka.ka_init(g, 2, 0.5, 1, R)
    ka.ka_observe_noalloc(s)   # waits for the initial state
    before = free_bytes()
    counts = ka.ka_observe(s)
    rows = ka.ka_run(s, [0, 0, 0])
    ka.ka_sweep(s, 0)
    # the counts take at most 18 KiB; 2 MiB is the largest unit that the runtime rounds up to
    assert before - free_bytes() <= 2 << 20
    for q in range(3):
        for a, b in zip(rows, counts[1:]):
            assert (a[q] == b).all()
    s.free()


# words drawn ahead would take 8 MiB
@pytest.mark.parametrize("size,R", [((2, 64), 64), ((2, 88), 128), ((2, 104), 64), ((3, 20), 128)])
def test_short_run_draws_in_its_sweeps(size, R):
    g = ka.ka_graph_lattice(*size)
    s = ka.ka_init(g, 2, 0.5, 1, R)
    ka.ka_observe_noalloc(s)
    before = free_bytes()
    ka.ka_run(s, [1])
    # three small buffers, each rounded up to 2 MiB at most
    assert before - free_bytes() <= 6 << 20
    s.free()
