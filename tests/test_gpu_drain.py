"""The guard queue's drain inside the pair loop: so many records per wavefront
that its segment of the queue (128 entries, drained from 64 on) would overflow,
by plans that do not split the records.  Every arrival lies in the window, so a
wavefront queues about records x histograms x guard width / wavefronts pairs;
the test asserts that this fills the segment one and a half times over before
it compares the sampled histograms with the oracle."""
import numpy as np
import pytest

import host_plans
import oracle
import scenes
from gpu_helpers import assert_parity_model, parity_tolerance, to_gpu

pytestmark = pytest.mark.gpu

# scan, lasers, bins, two units per workgroup
CASES = [((17, 64), None, 2000, True), ((24, 16), None, 9000, False), ((12, 31), (3, 3), 1000, True),
         ((12, 13), (2, 2), 9000, False)]


@pytest.mark.parametrize("scan,laser,T,pair", CASES)
def test_drain_inside_the_loop(scan, laser, T, pair):
    import torch
    import paper_2506_03747_amd as nl
    sc = scenes.tiny(seed=970, scan=scan, laser=laser, patches=(320, 330), n_bins=T, bin_ps=12000.0 / T, fwhm_ps=60.0,
                     half=0.5, zlo=0.3, zhi=0.9, masked=False)
    prm = nl.params_of(sc)
    plan = host_plans.forward_plan(prm, sc.n_patch_total)
    assert plan["n_split"] == 1 and plan["n_windows"] == 1 and plan["pair"] == int(pair)
    depth, albedo, mask = to_gpu(sc)
    tau, rec, n = nl.simulate(prm, depth, sc.patch_grid, albedo, mask)
    torch.cuda.synchronize()
    slots = plan["tl"] * plan["tx"] * plan["ty"] * (2 if pair else 1)
    waves = (plan["one"] or 1024) // 64
    guard = 32.0 * (T + 2) / 2 ** 24
    assert int(n.item()) * slots * guard / waves > 1.5 * 128
    H = sc.n_laser * sc.n_scan
    sub = np.sort(np.random.default_rng(970).choice(H, 48, replace=False)).astype(np.int32)
    records = oracle.patches(sc)
    ref = oracle.forward(sc, records, subset=sub)["tau"]
    got = tau.reshape(H, -1)[torch.from_numpy(sub).long().cuda()].cpu().numpy()
    assert_parity_model(got, ref, parity_tolerance(sc, ref, subset=sub, rec=records), what=f"drain {plan}")
