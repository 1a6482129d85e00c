"""The light-cone route summed by samples, at the sizes where it can go
wrong: cone layers at a tie, points that leave a piece of scan points partly
past the grid, one bin and one point, the longest rows (one and two rounds of
threads), and the thin, wide volumes that still go through the transforms.

Reference: the oracle's own pieces (volume samples, cone, time resampling,
taps) in fp64, the convolution as the sum over pixels that Eq. (3)-(5) define
and the resampling by its at most three coarse samples, so that rows of 16384
bins need no dense matrix.  Tolerance per histogram: fp32 rounding of the
output, 2^-24 relative, and the fixed-point rounding of the weights, below
1e-12 of the largest; 1e-6 covers both with room.  (The transforms are held to
the oracle's bar of 1e-5.)"""
import numpy as np
import pytest

from gpu_helpers import to_gpu
from oracle import lct as lct_oracle
from pins_lct import lct_scene

pytestmark = pytest.mark.gpu


def _reference(sc):
    N, M = sc.relay["nx"], sc.n_bins
    dt = sc.bin_ps * 1e-12
    dz = lct_oracle.C_LIGHT * dt / 2.0
    cone = np.roll(lct_oracle.psf(N, M, sc.relay["half_x"] / (M * lct_oracle.C_LIGHT * dt)), (N, N), (0, 1))
    V = lct_oracle.volume(sc.depth, sc.albedo, sc.mask, M, dz)
    conv = np.zeros((N, N, M))
    for x, y, j in zip(*np.nonzero(V)):
        J = j + 1
        c = (J * J - 1) // M
        # offsets (x' - x, y' - y) of the N x N points, from the cone centred at (N, N)
        part = cone[N - x:2 * N - x, N - y:2 * N - y, :M - c]
        conv[:, :, c:] += part * (V[x, y, j] / J / M)
    j = np.arange(M, dtype=np.int64)
    lo, hi = j * j, (j + 1) ** 2
    tau = np.zeros_like(conv)
    for s in range(3):
        c = lo // M + s
        ov = np.minimum(hi, (c + 1) * M) - np.maximum(lo, c * M)
        use = ov > 0
        tau[:, :, use] += conv[:, :, c[use]] * (ov[use] / (2.0 * j[use] + 1.0))
    tau /= ((j + 1) * dz) ** 3
    k = lct_oracle.taps(sc.fwhm_ps, sc.bin_ps)
    R = len(k) // 2
    pad = np.pad(tau, ((0, 0), (0, 0), (R, R)))
    return sum(k[i] * pad[:, :, 2 * R - i:2 * R - i + M] for i in range(2 * R + 1))


def _run(sc):
    import torch
    import paper_2506_03747_amd as nl
    depth, albedo, mask = to_gpu(sc)
    tau = nl.lct_forward(nl.params_of(sc), depth, albedo, mask)
    again = nl.lct_forward(nl.params_of(sc), depth, albedo, mask)
    torch.cuda.synchronize()
    return tau.cpu().numpy().astype(np.float64), torch.equal(tau, again)


SIZES = [dict(N=16, M=64, bin_ps=100.0, half=64 * lct_oracle.C_LIGHT * 100e-12 * 0.25, zlo=0.1, zhi=0.6, fwhm_ps=0.0),
         dict(N=13, M=128, bin_ps=64.0),
         dict(N=1, M=1, bin_ps=4000.0, zlo=0.3, zhi=0.4, masked=False, fwhm_ps=0.0),
         dict(N=90, M=64, bin_ps=120.0),
         dict(N=5, M=8192, bin_ps=1.0, zlo=0.2, zhi=0.9, fwhm_ps=40.0, masked=False),
         dict(N=3, M=16384, bin_ps=0.5, zlo=0.2, zhi=0.9, fwhm_ps=31.0, masked=False)]


@pytest.mark.parametrize("kw", SIZES, ids=[f"{k['N']}x{k['M']}" for k in SIZES])
def test_lct_by_samples(kw):
    sc = lct_scene(seed=11, **kw)
    if kw["N"] == 16:
        cone = lct_oracle.psf(16, 64, 0.25)
        assert (cone.sum(axis=2) == 2).any(), "the first size is there for its ties"
    ref = _reference(sc)
    got, same = _run(sc)
    assert same, "integer sums: the same bits on every run"
    r, g = ref.reshape(-1, sc.n_bins), got.reshape(-1, sc.n_bins)
    nr = np.linalg.norm(r, axis=1)
    assert np.all(np.linalg.norm(g - r, axis=1) <= 1e-6 * np.maximum(nr, 1e-9 * nr.max()))


def test_lct_thin_volume_by_transforms():
    sc = lct_scene(N=64, M=2, bin_ps=4000.0, seed=12, zlo=0.3, zhi=0.9)
    ref = lct_oracle.forward(sc)
    got, _ = _run(sc)
    assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)


def test_lct_empty_and_infinite():
    sc = lct_scene(N=16, M=64, bin_ps=100.0, seed=13, zlo=0.1, zhi=0.6)
    sc.mask[:] = 0
    assert not _run(sc)[0].any()
    sc.mask[:] = 1
    sc.albedo[3, 4] = np.inf
    assert np.isnan(_run(sc)[0]).all()
