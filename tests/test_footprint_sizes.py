"""ka_footprint against a count of its own of the arrays that a lattice sim allocates: state, words
drawn ahead, snapshots or a second copy of n.  Sizes include those where one class's words padded to
1024 threads would exceed the 8 MiB budget while the words themselves do not.  With a device present, the
library also knows which instances fit in LDS, so the same sizes run there too."""
import pytest

from paper_1710_05155_amd import ka

MIB = 1 << 20


def allocated(d, L, W):
    N = L ** d
    P = N // 4 ** d
    total = 3 * N * W * 8
    resident = P <= (512 if d == 2 else 128)
    if d == 3 and not resident:
        return total
    per_sweep = (4 * 8 if d == 2 else 16 * 12) * P * W * 8   # edges of a sweep x words
    sweeps = min(5461, 8 * MIB // per_sweep)
    # planes that a workgroup keeps in LDS draw in the sweep in 2D, and ahead from ten sweeps on in 3D
    if d == 3:
        in_lds = P < 64 or P == 64 and W > (28 if W % 2 else 256)
    elif P > 512:
        in_lds = P <= 576 and W % 2 and W >= 61
    else:
        in_lds = 9 <= P <= (144 if W > 256 else 100) and P * W * W >= 10 ** 6
    if not (in_lds and d == 2) and sweeps >= ((10 if in_lds and P > 1 else 3) if resident else 1):
        total += sweeps * per_sweep
    row = 2 * N * W * 8
    total += 4 * MIB // row * row if resident else N * W * 8
    return total


SIZES = [(2, 4, 1), (2, 4, 129), (2, 12, 129), (2, 32, 1), (2, 32, 129), (2, 64, 4), (2, 88, 2), (2, 92, 43), (2, 96, 45), (2, 96, 61), (2, 512, 1),
         (2, 512, 16), (2, 1024, 4), (3, 4, 3), (3, 12, 1), (3, 12, 90), (3, 16, 2), (3, 20, 1), (3, 20, 43), (3, 24, 4), (3, 128, 4)]


def check(d, L, W):
    footprint = ka.ka_footprint(ka.ka_graph_lattice(d, L), 64 * W)
    most = allocated(d, L, W)
    assert most <= footprint
    if d == 3 and L >= 24:   # above it only counts, thresholds, and the observation buffer that state copies leave (256 KiB)
        assert footprint <= most + 64 * W * 100 + (512 << 10)


@pytest.mark.parametrize("d,L,W", SIZES)
def test_footprint_holds_every_array(d, L, W):
    check(d, L, W)


@pytest.mark.gpu
@pytest.mark.parametrize("d,L,W", SIZES)
def test_footprint_holds_every_array_with_a_device(d, L, W):
    check(d, L, W)
