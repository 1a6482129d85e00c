"""Requests with few scan points and thousands of records in ticks and batched
calls, where no unit shape gives a request its share of workgroups: the same
bits as the calls alone wherever those do not split the patches."""
import numpy as np
import pytest

import scenes
from gpu_helpers import assert_parity, to_gpu

pytestmark = pytest.mark.gpu


def case(seed, scan, patches, T):
    return dict(seed=seed, scan=scan, patches=patches, n_bins=T, bin_ps=8000.0 / T * 1.5, fwhm_ps=60.0, half=0.8,
                zlo=0.3, zhi=0.9)


LISTS = [[case(960, (16, 16), (128, 128), 512)], [case(961, (13, 17), (128, 128), 512)],
         [case(962, (20, 20), (100, 90), 2048)], [case(963, (25, 22), (84, 19), 895)],
         [case(964, (3, 2), (150, 150), 700), case(965, (12, 12), (96, 96), 300)],
         [case(966, (8, 8), (128, 128), 512), case(967, (5, 9), (60, 70), 4000), case(968, (30, 31), (40, 50), 640)]]


@pytest.mark.parametrize("i", range(len(LISTS)))
def test_lists_match_calls_alone(i):
    import torch
    import paper_2506_03747_amd as nl
    scs = [scenes.tiny(**kw) for kw in LISTS[i]]
    reqs, alone = [], []
    for sc in scs:
        depth, albedo, mask = to_gpu(sc)
        reqs.append(dict(params=nl.params_of(sc), grid=sc.patch_grid, depth=depth, albedo=albedo, mask=mask))
        alone.append(nl.simulate(nl.params_of(sc), depth, sc.patch_grid, albedo, mask))
    slot = nl.TickGraph(len(scs), sum(sc.n_patch_total for sc in scs))
    got = [g[0] for g in slot.plan(reqs)]
    slot.launch()
    batched = nl.forward_batched([(nl.params_of(sc), rec, n, None) for sc, (_, rec, n) in zip(scs, alone)])
    torch.cuda.synchronize()
    for sc, (ref, _, _), tick, batch in zip(scs, alone, got, batched):
        for what, out in (("tick", tick), ("batched", batch)):
            if nl.get_plan(nl.params_of(sc), sc.n_patch_total)["n_split"] > 1:
                assert_parity(out.cpu().numpy(), ref.cpu().numpy().astype(np.float64), tol=1e-6, what=f"{what} {sc.name}")
            else:
                assert torch.equal(out.view(torch.int32), ref.view(torch.int32)), (what, sc.name)
    slot.close()
