"""The plans that the library's host side chooses, without a GPU."""
import ctypes as C
import random

import pytest

import host_plans
from host_plans import adjoint_plan, forward_plan, params, smooth_plan


def _problems(n, seed):
    rng = random.Random(seed)
    for _ in range(n):
        lasers = (rng.randint(1, 4), rng.randint(1, 4)) if rng.random() < 0.3 else (0, 0)
        yield (params(int(2 ** rng.uniform(0, 6.5)), int(2 ** rng.uniform(0, 6.5)), int(2 ** rng.uniform(5, 14.5)),
                      bin_ps=rng.uniform(2.0, 16.0), laser=lasers), int(2 ** rng.uniform(0, 18)))


def test_lists_split_only_where_the_call_alone_does():
    """A request in a list (any share of the GPU) has its patches split over
    workgroups only where the call alone has: elsewhere both give the same bits."""
    seen = 0
    for prm, n in _problems(400, 1):
        alone = forward_plan(prm, n)
        for target in (1, 3, 17, 60, 85, 128, 200, 256):
            got = forward_plan(prm, n, target, solo=False)
            assert got["one"] == 0 and got["n_windows"] == alone["n_windows"]
            assert alone["n_split"] > 1 or got["n_split"] == 1, (prm.relay.nx, prm.relay.ny, prm.n_bins, n, target)
            seen += got["n_split"] > 1
    assert seen > 20
    one = params(16, 16, 512)
    assert forward_plan(one, 128 * 128)["n_split"] == 1
    assert forward_plan(one, 128 * 128, 256, solo=False)["n_split"] == 1


def test_tuned_unit_that_does_not_fit_leaves_the_plan():
    """A tuning entry whose unit does not fit in LDS twice changes nothing: a
    call alone and a list's request take the plans they take without it."""
    nat = host_plans._native
    prm = params(18, 17, 1400)                   # two units of 4 x 2 histograms need more than 160 KB
    plans = [dict(solo=True), dict(solo=False), dict(target=40, solo=False)]
    want = [forward_plan(prm, 30000, **kw) for kw in plans]
    L = host_plans.lib()
    try:
        for unit in ((1, 4, 4), (1, 4, 2)):
            tab = (nat.TuningEntry * 1)(nat.TuningEntry(1, 1, 1 << 20, 1, 1 << 40, *unit))
            assert L.nlos_set_tuning(tab, 1) == 0
            assert [forward_plan(prm, 30000, **kw) for kw in plans] == want
        tab = (nat.TuningEntry * 1)(nat.TuningEntry(1, 1, 1 << 20, 1, 1 << 40, 1, 2, 1))
        assert L.nlos_set_tuning(tab, 1) == 0
        got = forward_plan(prm, 30000)
        assert (got["tx"], got["ty"], got["pair"]) == (2, 1, 1)
    finally:
        L.nlos_set_tuning(None, 0)


# scan, bins, ps per bin, FWHM in ps, records -> by moments (measured faster by more than a tenth)
SMOOTH_ROUTES = [((48, 40), 1024, 8.0, 50.0, 256, False), ((48, 40), 1600, 5.0, 60.0, 64, False),
                 ((100, 100), 1400, 8.0, 25.0, 1024, False), ((100, 100), 3000, 3.0, 50.0, 576, False),
                 ((20, 20), 2048, 4.0, 60.0, 16, False), ((48, 40), 1400, 8.0, 25.0, 2304, False), ((100, 100), 700, 6.0, 70.0, 64, True),
                 ((48, 40), 700, 6.0, 70.0, 1024, True), ((8, 8), 1024, 8.0, 50.0, 16, True),
                 ((48, 40), 1600, 5.0, 60.0, 4096, True), ((128, 128), 1024, 8.0, 50.0, 16384, True)]
ADJOINT_ROUTES = [((8, 8), 300, 16.0, 46.0, 4096, False), ((20, 20), 1024, 8.0, 50.0, 256, False),
                  ((100, 100), 1400, 8.0, 25.0, 1024, False), ((48, 40), 300, 16.0, 46.0, 256, False),
                  ((100, 100), 700, 6.0, 70.0, 16, True), ((48, 40), 1600, 5.0, 60.0, 2304, True),
                  ((100, 100), 400, 8.0, 50.0, 256, True), ((128, 128), 1024, 8.0, 50.0, 16384, True)]


@pytest.mark.parametrize("scan,T,bin_ps,fwhm_ps,n,moments", SMOOTH_ROUTES)
def test_smooth_forward_route(scan, T, bin_ps, fwhm_ps, n, moments):
    """Few records: the taps' work per pair is less than the moments' per bin."""
    assert (smooth_plan(params(*scan, T, bin_ps, fwhm_ps), n)["moments"] > 0) == moments


@pytest.mark.parametrize("scan,T,bin_ps,fwhm_ps,n,moments", ADJOINT_ROUTES)
def test_adjoint_route(scan, T, bin_ps, fwhm_ps, n, moments):
    """Few records or scan points: no pass of correlations over every row."""
    plan = adjoint_plan(params(*scan, T, bin_ps, fwhm_ps), n)
    assert (plan["moments"] > 0) == moments
    assert (plan["head_bytes"] > 0) == moments


@pytest.mark.parametrize("nx,points", [(1, 1), (2, 2), (3, 3), (4, 3), (50, 3)])
def test_smooth_points_per_workgroup_exist(nx, points):
    """Short rows leave room for three scan points per workgroup; a narrow scan
    gets no more than it has along x."""
    plan = smooth_plan(params(nx, 4000 // nx, 400, 8.0, 50.0), 5000)
    assert plan["moments"] == 6 and plan["tx"] == points


def test_adjoint_workspace_is_bounded():
    """The correlations' share of the workspace stays within 4 GiB however
    many scan points there are (the rest is the records' partials)."""
    nat = host_plans._native
    for scan, T, fwhm in (((512, 512), 2048, 83.0), ((2000, 1000), 1024, 50.0), ((256, 256), 3300, 160.0)):
        prm = params(*scan, T, 8.0, fwhm)
        plan = adjoint_plan(prm, 10000)
        assert plan["moments"] and plan["head_bytes"] <= (4 << 30) + (1 << 20), plan
        need = C.c_size_t(0)
        assert nat.lib().nlos_adjoint_workspace_bytes(C.byref(prm), 10000, C.byref(need)) == 0
        assert need.value == plan["head_bytes"] + plan["split"] * 10000 * 40


@pytest.mark.parametrize("scan,T", [((2050, 2050), 1000), ((4096, 4096), 100), ((2048, 2047), 1000)])
def test_smooth_launch_holds_every_scan(scan, T):
    """One launch has fewer than 2^32 threads: scans whose moment rows would need
    more workgroups of 1024 than that allows go by taps."""
    plan = smooth_plan(params(*scan, T, 8.0, 50.0), 5000)
    assert plan["workgroups"] * 1024 < 1 << 32
    assert (plan["moments"] > 0) == (scan == (2048, 2047))


@pytest.mark.parametrize("n,launches", [(1, 1), ((1 << 21) - 1, 1), (1 << 33, 1), (1 << 35, 2), (70 << 30, 3)])
def test_noise_launches_hold_every_array(n, launches):
    """An array of any size that fits the card is drawn in launches of fewer than
    2^32 threads each."""
    f = host_plans.lib().host_noise_launches
    f.restype = C.c_int64
    threads = C.c_int64(0)
    assert f(C.c_int64(n), C.byref(threads)) == launches
    assert 0 < threads.value < 1 << 32
