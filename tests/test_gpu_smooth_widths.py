"""Smooth forward and record adjoint at the widths and lengths where the plan
changes: the edges of each class of polynomial terms (sigma = 1.2, 1.6, 2.5,
4.9 bins) and a wide jitter, the longest rows of each layout of the forward's
LDS and one bin more, rows past the LDS (by taps), T not a multiple of 4 and
T below the support; walls with a partly filled last group of scan points.
Against the fp64 oracle, with the bars of the other smooth tests."""
import math

import numpy as np
import pytest

import oracle
from gpu_helpers import assert_parity, to_gpu
from pins_smooth import smooth_scene
from test_gpu_smooth import _assert_record_grads

pytestmark = pytest.mark.gpu


def fwhm(sigma, bin_ps):
    return sigma * bin_ps * 2.0 * math.sqrt(2.0 * math.log(2.0))


def case(seed, sigma, T, **kw):
    # bins so that the arrivals, at 3.3 to 6 ns, cross most of the window
    bin_ps = max(2.0, 6200.0 / T)
    return dict(seed=seed, n_bins=T, bin_ps=bin_ps, fwhm_ps=fwhm(sigma, bin_ps), **kw)


CASES = [
    case(701, 1.1999, 300), case(702, 1.2001, 300), case(703, 1.5999, 300), case(704, 1.6001, 301),
    case(705, 2.4999, 300), case(706, 2.5001, 302), case(707, 4.8999, 300), case(708, 4.9001, 303),
    case(709, 30.0, 640, scan=(4, 2)),                    # radius 180, T + 2 Rs = 1000
    case(710, 8.0, 40, scan=(2, 3)),                      # the support is longer than the window
    # radius 16, 6 terms: rows of 564 (three points), 565 (two), 848, 849 (one), 1696, 1697
    # (one workgroup per CU), 3402, 3403 (by taps)
    case(711, 2.65, 532, scan=(4, 3)), case(712, 2.65, 533, scan=(5, 2)), case(713, 2.65, 816, scan=(3, 2)),
    case(714, 2.65, 817), case(715, 2.65, 1664, scan=(2, 2)), case(716, 2.65, 1665, scan=(2, 2)),
    case(717, 2.65, 3370, scan=(2, 1)), case(718, 2.65, 3371, scan=(2, 1)),
    case(719, 1.9, 460, scan=(4, 4), cosines=False, standoff_m=0.4),
    # patches split over workgroups, several blocks of 4096 records in the adjoint
    case(720, 3.3, 900, scan=(3, 2), patches=(90, 70)),
]


@pytest.mark.parametrize("kw", CASES, ids=[str(k["seed"]) for k in CASES])
def test_smooth_widths(kw):
    import torch
    import paper_2506_03747_amd as nl
    sc = smooth_scene(**kw)
    depth, albedo, mask = to_gpu(sc)
    rec, n = nl.patches_from_depth(depth, sc.patch_grid, albedo, mask, cosines=sc.cosines)
    prm = nl.params_of(sc)
    tau = nl.forward_smooth(prm, rec, n)
    G = np.random.default_rng(kw["seed"]).standard_normal((sc.n_scan, sc.n_bins)).astype(np.float32)
    gr = nl.adjoint(prm, rec, n, torch.from_numpy(G).cuda())
    torch.cuda.synchronize()
    assert_parity(tau.cpu().numpy(), oracle.forward_smooth(sc), what=f"smooth {kw}")
    k = int(n.item())
    idx = rec[:k].cpu().numpy()[:, 7].view(np.int32)
    want = oracle.adjoint_records(sc, G.astype(np.float64))[idx]
    _assert_record_grads(gr[:k].cpu().numpy().astype(np.float64), want, f"adjoint {kw['seed']}")
    assert not gr[k:].cpu().numpy().any()


def test_adjoint_keeps_to_its_support():
    """An infinite upstream value reaches the records within the support of its
    bin and no others."""
    import torch
    import paper_2506_03747_amd as nl
    sc = smooth_scene(730, scan=(1, 1), patches=(20, 20), n_bins=512, bin_ps=12.0, fwhm_ps=fwhm(2.6, 12.0))
    depth, albedo, mask = to_gpu(sc)
    rec, n = nl.patches_from_depth(depth, sc.patch_grid, albedo, mask)
    prm = nl.params_of(sc)
    k = int(n.item())
    bins = nl.debug_bins(prm, rec, n)[0, :k].cpu().numpy()
    at = int(np.sort(bins)[k // 3])
    G = torch.zeros((1, sc.n_bins), device="cuda")
    G[0, at] = float("inf")
    gr = nl.adjoint(prm, rec, n, G)[:k].cpu().numpy()
    rs = math.ceil(6 * 2.6)
    away = np.abs(bins - at) > rs
    assert away.any() and not away.all()
    assert np.isfinite(gr[away]).all() and not gr[away].any()
    assert not np.isfinite(gr[~away][:, 3]).any()


def test_smooth_without_records():
    import torch
    import paper_2506_03747_amd as nl
    prm = nl.make_params(dict(nx=3, ny=2, half_x=0.5, half_y=0.5), 200, 10.0, 60.0)
    rec = torch.empty((0, 8), device="cuda")
    assert not nl.forward_smooth(prm, rec).any()
