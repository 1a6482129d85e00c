"""The plan a call alone takes (one or two units per workgroup, whole and half
workgroups, split patches) against the paired plan of every unit shape named
by a tuning table: the same bits wherever neither splits the patches, and the
oracle's histograms.  Sizes on both sides of what the plans depend on: a
histogram, a unit or a pair of units that just fits in LDS, fewer and more
workgroups than CUs, odd grids, lasers."""
import pytest

import oracle
import scenes
from gpu_helpers import assert_parity, gpu_forward, to_gpu

pytestmark = pytest.mark.gpu

CONF_UNITS = [(1, 4, 4), (1, 4, 2), (1, 2, 2), (1, 2, 1), (1, 1, 1)]
NC_UNITS = [(2, 2, 2), (2, 1, 2), (1, 1, 2), (1, 1, 1)]


def case(scan, patches, T, **kw):
    # window of 2.4 m one way: most arrivals inside, those of far pairs past it
    return dict(scan=scan, patches=patches, n_bins=T, bin_ps=8000.0 / T * 1.5, fwhm_ps=60.0, half=0.8, zlo=0.3,
                zhi=0.9, **kw)


CASES = [case((1, 1), (40, 30), 256), case((3, 5), (33, 17), 777), case((61, 47), (40, 31), 333),
         case((37, 29), (24, 20), 1130), case((33, 33), (24, 20), 1200), case((20, 20), (24, 20), 2300),
         case((18, 17), (24, 20), 2380), case((9, 11), (24, 20), 4700), case((7, 6), (24, 20), 9000),
         case((130, 67), (12, 10), 500), case((34, 33), (30, 20), 601, cosines=False),
         case((9, 7), (24, 20), 900, laser=(3, 3)), case((24, 23), (20, 20), 1150, laser=(3, 2)),
         case((17, 16), (20, 20), 2300, laser=(2, 3)), case((8, 9), (20, 20), 4700, laser=(1, 3), standoff_m=0.5),
         case((64, 62), (100, 90), 1024), case((16, 32), (120, 120), 1500), case((128, 33), (60, 60), 2048),
         case((30, 31), (100, 90), 2048, laser=(3, 3)), case((33, 40), (200, 180), 640),
         case((2, 2), (300, 310), 300), case((2, 1), (130, 130), 700, laser=(2, 1))]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_own_plan_matches_paired_units(i):
    import torch
    import paper_2506_03747_amd as nl
    sc = scenes.tiny(seed=900 + i, **CASES[i])
    prm = nl.params_of(sc)
    n_rec = sc.patch_grid["nx"] * sc.patch_grid["ny"]
    ref = oracle.forward(sc)["tau"]
    nl.set_tuning([])
    try:
        own = nl.get_plan(prm, n_rec)
        assert own["pair"] == 1 and own["n_windows"] == 1
        tau, _, _ = gpu_forward(sc)
        assert_parity(tau.cpu().numpy(), ref, what=f"own plan {own}")
        depth, albedo, mask = to_gpu(sc)
        one = nl.simulate(prm, depth, sc.patch_grid, albedo, mask)[0]
        if own["n_split"] == 1:
            assert torch.equal(one, tau)
        else:
            assert_parity(one.cpu().numpy(), tau.cpu().numpy().astype("f8"), tol=1e-6, what="one call")
        for unit in NC_UNITS if sc.laser is not None else CONF_UNITS:
            nl.set_tuning([dict(confocal=int(sc.laser is None), t_min=1, t_max=1 << 20, h_min=1, h_max=1 << 40,
                                tl=unit[0], tx=unit[1], ty=unit[2])])
            plan = nl.get_plan(prm, n_rec)
            if (plan["tl"], plan["tx"], plan["ty"]) != unit:
                continue                    # two of these units do not fit in LDS
            forced, _, _ = gpu_forward(sc)
            if plan["n_split"] == 1 and own["n_split"] == 1:
                assert torch.equal(forced, tau), (own, plan)
            else:
                assert_parity(forced.cpu().numpy(), tau.cpu().numpy().astype("f8"), tol=1e-6, what=f"unit {unit}")
    finally:
        nl.reset_tuning()


def test_many_records_per_wavefront():
    """A wavefront's guard queue fills and is drained several times."""
    import torch
    import paper_2506_03747_amd as nl
    sc = scenes.tiny(seed=950, scan=(2, 2), patches=(300, 300), n_bins=4000, bin_ps=3.0, fwhm_ps=20.0, half=0.8,
                     zlo=0.3, zhi=0.9)
    depth, albedo, mask = to_gpu(sc)
    prm = nl.params_of(sc)
    nl.set_tuning([dict(confocal=1, t_min=1, t_max=1 << 20, h_min=1, h_max=1 << 40, tl=1, tx=2, ty=1)])
    try:
        tau = nl.simulate(prm, depth, sc.patch_grid, albedo, mask)[0]
        assert_parity(tau.cpu().numpy(), oracle.forward(sc)["tau"], what="many records")
    finally:
        nl.reset_tuning()
    assert torch.isfinite(tau).all()
