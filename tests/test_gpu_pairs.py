"""Four-point sums against the autocorrelations of the exported state (FFT per replica, rounded to
integers): tiles of one and several rows, rows beyond the lattice, word counts that are not a multiple of the
words a tile holds, radii up to half the lattice (where a displacement is its own opposite), and
radii whose halo does not fit in LDS."""
import numpy as np
import pytest

from paper_1710_05155_amd import ka

pytestmark = pytest.mark.gpu


def shells(d, L, r2_max):
    c = (np.arange(L) + L // 2 - 1) % L - (L // 2 - 1)      # minimum image, L/2 positive
    c = np.where(c == -(L // 2), L // 2, c)
    r2 = sum(np.meshgrid(*([c * c] * d), indexing="ij"))
    return np.where(r2 <= r2_max, r2, -1).ravel()


def sums(n, n0, d, L, R, r2_max):
    shape = (L,) * d
    r2 = shells(d, L, r2_max)
    keep = r2 >= 0
    S2 = np.zeros(r2_max + 1, dtype=np.int64)
    total = np.zeros(L ** d)
    corr = np.zeros(L ** d)
    for b in range(R):
        q = (((n[b >> 6] & n0[b >> 6]) >> np.uint64(b & 63)) & np.uint64(1)).astype(float)
        total += q
        f = np.fft.fftn(q.reshape(shape))
        corr += np.rint(np.fft.ifftn(f * f.conj()).real).ravel()
    f = np.fft.fftn(total.reshape(shape))
    prod = np.rint(np.fft.ifftn(f * f.conj()).real).ravel()
    S2 = np.bincount(r2[keep], corr[keep], r2_max + 1).astype(np.int64)
    S11 = np.bincount(r2[keep], prod[keep], r2_max + 1).astype(np.int64)
    return S2, S11, np.bincount(r2[keep], minlength=r2_max + 1)


@pytest.mark.parametrize("d,L,R,r2_max", [(2, 4, 64, 8), (2, 36, 128, 100), (2, 100, 320, 37), (2, 64, 64, 1024), (2, 132, 64, 1500),
                                          (2, 512, 64, 36), (3, 4, 1024, 12), (3, 12, 192, 36), (3, 20, 256, 300), (3, 36, 64, 36),
                                          (3, 36, 128, 0), (3, 64, 64, 2)])
def test_pair_sums_equal_autocorrelations(d, L, R, r2_max):
    s = ka.ka_init(ka.ka_graph_lattice(d, L), 2 * d - 2, 0.6, 17, R)
    ka.ka_sweep(s, 2)
    S2, S11, cnt = ka.ka_observe_pairs(s, r2_max)
    n, n0, _, _ = ka.ka_get_state(s)
    s.free()
    eS2, eS11, ecnt = sums(n, n0, d, L, R, r2_max)
    assert np.array_equal(cnt, ecnt)
    assert np.array_equal(S2, eS2)
    assert np.array_equal(S11, eS11)
