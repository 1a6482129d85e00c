"""Records of small maps, made by one launch, at its edges: one pixel, one row,
odd blocks, exactly 16 blocks of 256 pixels and one more (two launches), maps
with no, one or all pixels present, with non-finite and non-positive depths;
against the oracle's records, and the one-call path (whose summaries the same
launch makes) against the two calls, bit for bit."""
import numpy as np
import pytest

import oracle
import scenes
from gpu_helpers import to_gpu

pytestmark = pytest.mark.gpu

CASES = [((1, 1), "all"), ((1, 37), "some"), ((16, 16), "all"), ((17, 15), "some"), ((63, 65), "some"),
         ((64, 64), "all"), ((64, 64), "none"), ((64, 64), "one"), ((256, 16), "some"), ((257, 15), "some"),
         ((30, 31), "odd"), ((5, 200), "odd")]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_small_maps(i):
    import torch
    import paper_2506_03747_amd as nl
    shape, kind = CASES[i]
    sc = scenes.tiny(seed=600 + i, scan=(6, 5), patches=shape, n_bins=200, bin_ps=30.0)
    rng = np.random.default_rng(i)
    if kind == "all":
        sc.mask[:] = 1
    elif kind == "none":
        sc.mask[:] = 0
    elif kind == "one":
        sc.mask[:] = 0
        sc.mask[41, 62] = 1
    elif kind == "odd":
        bad = rng.uniform(size=shape)
        sc.depth[bad < 0.05] = np.nan
        sc.depth[(bad >= 0.05) & (bad < 0.1)] = np.inf
        sc.depth[(bad >= 0.1) & (bad < 0.15)] = 0.0
        sc.albedo[(bad >= 0.15) & (bad < 0.2)] = 0.0
    depth, albedo, mask = to_gpu(sc)
    rec, n = nl.patches_from_depth(depth, sc.patch_grid, albedo, mask)
    present = (sc.mask != 0) & np.isfinite(sc.depth) & (sc.depth > 0) & (sc.albedo > 0)
    k = int(n.item())
    assert k == int(present.sum())
    got = rec[:k].cpu().numpy()
    np.testing.assert_array_equal(np.sort(got[:, 7].view(np.int32)), np.nonzero(present.ravel())[0])
    want = oracle.patches(sc)[got[:, 7].view(np.int32)]
    np.testing.assert_array_equal(got[:, :3], want[:, :3].astype(np.float32))
    if kind != "odd":   # (a non-finite neighbour leaves no normal)
        np.testing.assert_allclose(got[:, 3:7], want[:, 3:7], rtol=1e-5, atol=1e-6)
    prm = nl.params_of(sc)
    tau = nl.forward(prm, rec, n)
    one, rec1, n1 = nl.simulate(prm, depth, sc.patch_grid, albedo, mask)
    torch.cuda.synchronize()
    assert int(n1.item()) == k and torch.equal(rec1[:k].view(torch.int32), rec[:k].view(torch.int32))
    if kind != "odd":
        assert torch.equal(one, tau)
