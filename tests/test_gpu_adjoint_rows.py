"""The adjoint's correlation rows where the gradient is not read in whole
16-byte words: rows shorter than one such read and rows whose ends fall at
each place within one.  Against the fp64 oracle, with the bars of the other
smooth tests."""
import math

import numpy as np
import pytest

import oracle
from gpu_helpers import to_gpu
from pins_smooth import smooth_scene
from test_gpu_smooth import _assert_record_grads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,sigma", [(1, 1.3), (2, 1.3), (3, 2.0), (5, 1.3), (6, 2.0), (7, 3.0), (13, 2.0), (258, 6.0),
                                     (511, 12.0), (601, 2.6), (2049, 5.0)])
def test_unaligned_rows(T, sigma):
    import torch
    import paper_2506_03747_amd as nl
    bin_ps = 6200.0 / T
    sc = smooth_scene(seed=800 + T, n_bins=T, bin_ps=bin_ps, fwhm_ps=sigma * bin_ps * 2.0 * math.sqrt(2.0 * math.log(2.0)),
                      scan=(5, 3), patches=(31, 27))
    depth, albedo, mask = to_gpu(sc)
    rec, n = nl.patches_from_depth(depth, sc.patch_grid, albedo, mask, cosines=sc.cosines)
    G = np.random.default_rng(T).standard_normal((sc.n_scan, sc.n_bins)).astype(np.float32)
    gr = nl.adjoint(nl.params_of(sc), rec, n, torch.from_numpy(G).cuda())
    torch.cuda.synchronize()
    k = int(n.item())
    idx = rec[:k].cpu().numpy()[:, 7].view(np.int32)
    want = oracle.adjoint_records(sc, G.astype(np.float64))[idx]
    _assert_record_grads(gr[:k].cpu().numpy().astype(np.float64), want, f"adjoint T {T}")
    assert not gr[k:].cpu().numpy().any()
