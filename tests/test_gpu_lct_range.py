"""The light-cone route's fixed-point sums over a wide range of albedos, and the
two kinds of volumes that still go through the transforms: thin, wide ones and
rows past the LDS.

Reference of the first: the sum over pixels in fp64 at sampled scan points (the
oracle's cone, the oracle's time resampling).  Every bin of every sampled row is
compared by itself: a bin that only dim pixels reach must be right to the
rounding of the output and of a few fp64 operations, 2 x 2^-24, beside pixels
10^8 or 10^10 times brighter (all weights are positive: nothing cancels).  The
transforms are held to the oracle's bar of 1e-5."""
import numpy as np
import pytest

from gpu_helpers import to_gpu
from oracle import lct as lct_oracle
from pins_lct import lct_scene
from test_gpu_lct_samples import _reference, _run

pytestmark = pytest.mark.gpu


def _rows(sc, points):
    N, M = sc.relay["nx"], sc.n_bins
    dt = sc.bin_ps * 1e-12
    dz = lct_oracle.C_LIGHT * dt / 2.0
    cone = np.roll(lct_oracle.psf(N, M, sc.relay["half_x"] / (M * lct_oracle.C_LIGHT * dt)), (N, N), (0, 1))
    J = np.floor(np.asarray(sc.depth, np.float64) / dz).astype(np.int64) + 1
    w = 1.0 / J / M * np.asarray(sc.albedo, np.float64)
    assert (sc.mask is None or sc.mask.all()) and J.max() <= M
    c = (J * J - 1) // M
    j = np.arange(M, dtype=np.int64)
    lo, hi = j * j, (j + 1) ** 2
    out = []
    for x, y in points:
        part = cone[x + 1:x + N + 1, y + 1:y + N + 1, :M][::-1, ::-1]     # offset (x - px, y - py) of every pixel
        px, py, k = np.nonzero(part)
        conv = np.zeros(M)
        at = c[px, py] + k
        np.add.at(conv, at[at < M], w[px, py][at < M])
        tau = np.zeros(M)
        for s in range(3):
            b = lo // M + s
            ov = np.minimum(hi, (b + 1) * M) - np.maximum(lo, b * M)
            use = ov > 0
            tau[use] += conv[b[use]] * (ov[use] / (2.0 * j[use] + 1.0))
        out.append(tau / ((j + 1) * dz) ** 3)
    return np.array(out)


@pytest.mark.parametrize("N,M,bin_ps,dim", [(64, 512, 16.0, 1e-10), (128, 256, 30.0, 1e-10), (260, 128, 60.0, 1e-8)])
def test_dim_pixels_beside_bright_ones(N, M, bin_ps, dim):
    rng = np.random.default_rng(N)
    sc = lct_scene(N=N, M=M, bin_ps=bin_ps, seed=21, zlo=0.25, zhi=0.45, fwhm_ps=0.0, masked=False)
    bright = rng.random((N, N)) < 4.0 / (N * N)
    bright[1, 2] = True
    sc.albedo = np.where(bright, 1.0, dim * rng.uniform(0.5, 1.0, (N, N))).astype(np.float32)
    points = [(0, 0), (N - 1, N - 1), (1, 2)] + [tuple(p) for p in rng.integers(0, N, (13, 2))]
    want = _rows(sc, points)
    got, same = _run(sc)
    assert same
    got = np.array([got.reshape(N, N, M)[x, y] for x, y in points])
    assert ((want > 0) == (got > 0)).all()
    on = want > 0
    assert on.sum() > 16 * 20
    assert np.max(np.abs(got[on] / want[on] - 1.0)) <= 2.0 ** -23


def test_wide_volume_by_transforms():
    sc = lct_scene(N=160, M=16, bin_ps=500.0, seed=22, zlo=0.2, zhi=0.9)
    ref = lct_oracle.forward(sc)
    got, _ = _run(sc)
    assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)


def test_rows_past_the_lds_by_transforms():
    sc = lct_scene(N=3, M=32768, bin_ps=0.25, seed=23, zlo=0.2, zhi=0.9, fwhm_ps=15.0, masked=False)
    ref = _reference(sc)
    got, _ = _run(sc)
    r, g = ref.reshape(9, -1), got.reshape(9, -1)
    # (past the first bins, where the resampling amplifies the transforms' noise 10^9-fold)
    late = slice(2048, None)
    assert np.linalg.norm(g[:, late] - r[:, late]) <= 1e-5 * np.linalg.norm(r)
