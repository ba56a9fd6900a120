"""Ring Fourier transforms of map2alm at the sizes where its paths change:
Nside 4096 (8192-point transforms), Nside that are not powers of two (the
belt by the chirp transform), and the edges of the classes of transform
sizes.  Ring-sparse maps against numpy's FFT of each ring times the oracle's
lambda_lm, every a_lm within 1e-11 of max |a| (the bar of the full-size
ring-sparse test)."""
import numpy as np
import pytest

from helpers import ring_sparse_alm

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _length(nside, r):
    return 4 * min(r, nside, 4 * nside - r)


def _first(nside, r):
    N = nside
    if r < N:
        return 2 * r * (r - 1)
    if r <= 3 * N:
        return 2 * N * (N - 1) + (r - N) * 4 * N
    k = 4 * N - r
    return 12 * N * N - 2 * k * (k + 1)


@pytest.mark.parametrize("nside,lmax", [(4096, 150), (2048, 150), (250, 320), (256, 300),
                                        (257, 300), (300, 260), (1500, 130), (2049, 70),
                                        (4095, 70)])
def test_ring_sparse(nside, lmax):
    from paper_1204_5041_amd import binding as B
    N = nside
    rings = {1, 2, 3, 128, 129, 256, 257, 1024, 1025, 2048, 2049, N - 1, N, N + 1, 2 * N - 1,
             2 * N, 2 * N + 1, 3 * N - 1, 3 * N, 3 * N + 1, 4 * N - 257, 4 * N - 1}
    rings = sorted(r for r in rings if 1 <= r <= 4 * N - 1)
    rng = np.random.Generator(np.random.PCG64(nside))
    hmap = np.zeros(12 * N * N)
    for r in rings:
        hmap[_first(N, r):_first(N, r) + _length(N, r)] = rng.standard_normal(_length(N, r))
    ref = ring_sparse_alm(N, lmax, hmap, rings)
    print("ring-sparse map", nside, lmax, flush=True)
    got = B.map2alm(torch.from_numpy(hmap).cuda(), lmax).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= 1e-11 * np.max(np.abs(ref))


@pytest.mark.parametrize("nside,lmax", [(2, 3), (16, 40), (32, 64), (33, 70), (64, 100), (128, 300),
                                        (200, 30), (256, 512), (512, 600)])
def test_ring_pairs_per_lane(nside, lmax):
    """Every number of ring pairs per lane and degrees per group that the
    Legendre kernel takes, with one and several blocks of ring pairs, against
    the oracle's lambda_lm on a few rings (the same bar)."""
    from paper_1204_5041_amd import binding as B
    N = nside
    rings = sorted({1, N // 2 + 1, N, 2 * N - 1, 2 * N, 3 * N, 4 * N - 1})
    rng = np.random.Generator(np.random.PCG64(7 * nside))
    hmap = np.zeros(12 * N * N)
    for r in rings:
        hmap[_first(N, r):_first(N, r) + _length(N, r)] = rng.standard_normal(_length(N, r))
    ref = ring_sparse_alm(N, lmax, hmap, rings)
    got = B.map2alm(torch.from_numpy(hmap).cuda(), lmax).cpu().numpy()
    assert np.max(np.abs(got - ref)) <= 1e-11 * np.max(np.abs(ref))
