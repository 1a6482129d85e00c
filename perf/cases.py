"""Performance cases of the transient NLOS simulator.

Each case is one call, or one short sequence of calls, through the package's
public entry points, at sizes of its own workloads (the scene generators, the
benchmark, the tests) or generic ones:

  simulate     depth map -> jittered histograms, confocal or with a laser
               grid (one call, or records first and the forward after)
  smooth       the differentiable forward and its backward
  noise        Poisson noise on a jittered frame
  lct          the light-cone route
  tick         a list of mixed requests as one serving tick
"""
import math
import random

import torch

import paper_2506_03747_amd as nl

C_LIGHT = 299792458.0
_NAMES = ("nx", "ny", "half_x", "half_y", "cx", "cy")


def _sim(name, scan, maps, n_bins, bin_ps, fwhm_ps, half=1.0, standoff=0.0, laser=(0, 0), cosines=True,
         albedo=True, mask=True, zlo=0.4, zhi=1.2, calls=1):
    return dict(name=name, kind="simulate", sx=scan[0], sy=scan[1], px=maps[0], py=maps[1], n_bins=n_bins,
                bin_ps=bin_ps, fwhm_ps=fwhm_ps, half=half, standoff=standoff, lx=laser[0], ly=laser[1],
                cosines=cosines, albedo=albedo, mask=mask, zlo=zlo, zhi=zhi, calls=calls)


def _smooth(name, scan, maps, n_bins, bin_ps, fwhm_ps, mask=False, zlo=0.4, zhi=1.2):
    return dict(name=name, kind="smooth", sx=scan[0], sy=scan[1], px=maps[0], py=maps[1], n_bins=n_bins,
                bin_ps=bin_ps, fwhm_ps=fwhm_ps, half=1.0, standoff=0.0, lx=0, ly=0, cosines=True, albedo=True,
                mask=mask, zlo=zlo, zhi=zhi)


def _noise(name, scan, n_bins, nr_db, peak):
    return dict(name=name, kind="noise", sx=scan[0], sy=scan[1], px=64, py=64, n_bins=n_bins, bin_ps=8.0,
                fwhm_ps=50.0, half=1.0, standoff=0.0, lx=0, ly=0, cosines=True, albedo=True, mask=True,
                zlo=0.4, zhi=1.2, nr_db=nr_db, peak=peak)


def _lct(name, n, n_bins, bin_ps, fwhm_ps, mask=False, zlo=0.4, zhi=1.2):
    return dict(name=name, kind="lct", sx=n, sy=n, px=n, py=n, n_bins=n_bins, bin_ps=bin_ps, fwhm_ps=fwhm_ps,
                half=1.0, standoff=0.0, lx=0, ly=0, cosines=False, albedo=True, mask=mask, zlo=zlo, zhi=zhi)


def _tick(name, requests, mix, max_scan, max_patches):
    return dict(name=name, kind="tick", requests=requests, mix=mix, max_scan=max_scan, max_patches=max_patches)


def listed():
    return [
        # the smallest call, as a test or an interactive probe makes it: launches and the host count
        _sim("probe-8x8", (8, 8), (24, 31), 256, 16.0, 70.0, half=0.5, zlo=0.3, zhi=0.6),
        # a quick preview on a small wall, device legs included (the cfg1 scene's sizes)
        _sim("preview-32x32", (32, 32), (64, 64), 512, 16.0, 70.0, half=0.5, standoff=1.0, zlo=0.45, zhi=0.55),
        # the benchmark's headline step (cfg2)
        _sim("frame-64x64", (64, 64), (256, 256), 1024, 8.0, 50.0),
        # records made once and simulated after, sizes that divide nothing, Eq. (1) without cosines, no maps but depth
        _sim("ragged-61x47", (61, 47), (150, 201), 777, 11.3, 60.0, half=0.8, cosines=False, albedo=False,
             mask=False, calls=2),
        # the largest request of the serving mix (cfg4's upper ends)
        _sim("large-128x128", (128, 128), (512, 512), 2048, 8.0, 50.0, zlo=0.5, zhi=1.5),
        # a laser grid of a few points on a ragged detector grid
        _sim("lasers-3x2", (33, 29), (100, 90), 1000, 8.0, 45.0, laser=(3, 2), standoff=0.5),
        # the full non-confocal acquisition (cfg3)
        _sim("lasers-8x8", (128, 128), (128, 128), 2048, 4.0, 30.0, laser=(8, 8), standoff=2.0),
        # one optimisation step of a depth map against a measured volume (cfg5): forward and gradients
        _smooth("fit-128x128", (128, 128), (128, 128), 1024, 8.0, 50.0),
        # the same on a coarser scan with the fine bins and wide jitter of the serving mix's ranges, T not a multiple of 4
        _smooth("fit-48x40", (48, 40), (96, 80), 1501, 5.0, 60.0, mask=True, zlo=0.3, zhi=0.9),
        # photon noise on the headline frame, a few tens of counts at the peak
        _noise("noise-64x64", (64, 64), 1024, 2.0, 40.0),
        # the light-cone cross-check on the cfg5 scene
        _lct("cone-128", 128, 1024, 8.0, 50.0),
        # one tick of the serving loop: mixed requests of cfg4's ranges
        _tick("tick-8", 8, 4, 128, 262144),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["simulate", "simulate", "lasers", "smooth", "smooth", "noise", "lct", "tick"])
    if kind == "tick":
        c = _tick("", rng.randint(2, 10), rng.randrange(1 << 20), rng.randint(40, 128), _log(rng, 6000, 200000))
    elif kind == "lct":
        m = 2 ** rng.randint(7, 10)
        c = _lct("", _log(rng, 12, 128), m, 8192.0 / m, rng.uniform(30.0, 70.0) * 1024 / m, rng.random() < 0.5)
    elif kind == "noise":
        c = _noise("", (_log(rng, 8, 100), _log(rng, 8, 100)), rng.randint(200, 1200), rng.choice([0.0, 2.0, 5.0]),
                   math.exp(rng.uniform(0.0, math.log(400.0))))
    else:
        # window and depths as in the serving mix: arrivals land in the window
        n_bins = _log(rng, 256, 2048 if kind != "smooth" else 1536)
        bin_ps = rng.uniform(4.0, 16.0)
        reach = min(C_LIGHT * n_bins * bin_ps * 1e-12 / 2, 3.0)
        z = dict(zlo=max(0.1, 0.2 * reach), zhi=max(0.25, 0.6 * reach))
        fwhm = rng.uniform(30.0, 70.0)
        masked = rng.random() < 0.6
        if kind == "smooth":
            c = _smooth("", (_log(rng, 8, 100), _log(rng, 8, 100)), (_log(rng, 16, 128), _log(rng, 16, 128)), n_bins,
                        bin_ps, fwhm, masked, **z)
        else:
            opt = dict(half=rng.choice([0.5, 0.8, 1.0]), standoff=rng.choice([0.0, 0.0, 0.5, 1.0]),
                       cosines=rng.random() < 0.75, albedo=rng.random() < 0.75, mask=masked, calls=rng.choice([1, 1, 2]))
            if kind == "lasers":
                c = _sim("", (_log(rng, 12, 96), _log(rng, 12, 96)), (_log(rng, 24, 128), _log(rng, 24, 128)), n_bins,
                         bin_ps, fwhm, laser=(rng.randint(1, 6), rng.randint(1, 6)), **opt, **z)
            else:
                c = _sim("", (_log(rng, 6, 128), _log(rng, 6, 128)), (_log(rng, 16, 400), _log(rng, 16, 400)), n_bins,
                         bin_ps, fwhm, **opt, **z)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# Inputs

def _grid(nx, ny, half):
    return dict(zip(_NAMES, (nx, ny, half, half, 0.0, 0.0)))


def _params(c):
    laser = _grid(c["lx"], c["ly"], c["half"]) if c["lx"] else None
    return nl.make_params(_grid(c["sx"], c["sy"], c["half"]), c["n_bins"], c["bin_ps"], c["fwhm_ps"], c["standoff"],
                          laser=laser, cosines=c["cosines"])


def _field(gen, nx, ny, cells):
    """A smooth random field [nx, ny] in [0, 1], about `cells` features per axis."""
    g = torch.randn((1, 1, cells, cells), generator=gen, device="cuda")
    f = torch.nn.functional.interpolate(g, size=(nx, ny), mode="bicubic", align_corners=True)[0, 0]
    lo, hi = f.min(), f.max()
    return ((f - lo) / (hi - lo)).contiguous()


def _maps(c, seed):
    """depth, albedo, mask on the GPU: a smooth surface, uniform albedo, a blob of about half the pixels."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed) & 0x7FFFFFFF)
    nx, ny = c["px"], c["py"]
    depth = c["zlo"] + (c["zhi"] - c["zlo"]) * _field(gen, nx, ny, 7)
    albedo = torch.rand((nx, ny), generator=gen, device="cuda") if c["albedo"] else None
    mask = None
    if c["mask"]:
        f = _field(gen, nx, ny, 6)
        mask = (f > f.median()).to(torch.uint8)
    return depth.contiguous(), albedo, mask


def _requests(c):
    """The tick's requests as simulate cases: sizes of the serving mix, from the case's own number."""
    rng, got = random.Random(c["mix"]), []
    for _ in range(c["requests"]):
        n = rng.randint(32, c["max_scan"])
        p = max(2, round(math.sqrt(rng.randint(4096, c["max_patches"]))))
        n_bins, bin_ps = rng.choice([512, 1024, 2048]), rng.uniform(4.0, 16.0)
        half_path = C_LIGHT * n_bins * bin_ps * 1e-12 / 2
        got.append(_sim("", (n, n), (p, p), n_bins, bin_ps, rng.uniform(30.0, 70.0), zlo=0.2 * half_path,
                        zhi=0.6 * half_path))
    return got


def _upstream(c, seed):
    """The upstream gradient of a fit: a residual, white over the bins."""
    gen = torch.Generator(device="cuda").manual_seed((int(seed) + 77777) & 0x7FFFFFFF)
    return torch.randn((c["sx"], c["sy"], c["n_bins"]), generator=gen, device="cuda")


def prepare(case, seed):
    c = case
    if c["kind"] == "tick":
        reqs = []
        for i, r in enumerate(_requests(c)):
            depth, albedo, mask = _maps(r, seed * 1000 + i)
            prm = _params(r)
            reqs.append(dict(params=prm, grid=_grid(r["px"], r["py"], r["half"]), depth=depth, albedo=albedo,
                             mask=mask, out=torch.empty(nl.out_shape(prm), device="cuda"),
                             patches=torch.empty((r["px"] * r["py"], 8), device="cuda"),
                             n_active=torch.empty(1, dtype=torch.int32, device="cuda")))
        pixels = sum(r["depth"].numel() for r in reqs)
        return dict(kind="tick", requests=reqs, slots=[nl.TickGraph(len(reqs), pixels) for _ in range(2)], turn=0)
    depth, albedo, mask = _maps(c, seed)
    prm, grid = _params(c), _grid(c["px"], c["py"], c["half"])
    s = dict(kind=c["kind"], params=prm, grid=grid, depth=depth, albedo=albedo, mask=mask, cosines=c["cosines"],
             calls=c.get("calls", 1), whole=not c["mask"])
    if c["kind"] == "smooth":
        s["depth"].requires_grad_()
        s["albedo"].requires_grad_()
        s["upstream"] = _upstream(c, seed)
    elif c["kind"] == "noise":
        tau = nl.simulate(prm, depth, grid, albedo, mask)[0]
        # scaled so that the brightest bin expects `peak` photons: lambda = tau Var(tau) / 10^(nr / 10)
        lam = float(tau.max().double() * tau.double().var(correction=0)) / 10.0 ** (c["nr_db"] / 10.0)
        s.update(tau=tau * (c["peak"] / lam) ** (1.0 / 3.0) if lam > 0.0 else tau, nr_db=c["nr_db"], seed=int(seed))
    return s


def run(state):
    s = state
    if s["kind"] == "simulate":
        if s["calls"] == 2:
            rec, n = nl.patches_from_depth(s["depth"], s["grid"], s["albedo"], s["mask"], cosines=s["cosines"])
            tau = nl.forward(s["params"], rec, n)
        else:
            tau, rec, n = nl.simulate(s["params"], s["depth"], s["grid"], s["albedo"], s["mask"])
        # (without a mask every record is written)
        return {"tau": tau, "n_active": n, "records": rec if s["whole"] else None}
    if s["kind"] == "smooth":
        tau = nl.smooth_transient(s["depth"], s["albedo"], s["grid"], s["params"], s["mask"])
        gd, ga = torch.autograd.grad(tau, (s["depth"], s["albedo"]), s["upstream"])
        return {"tau": tau, "grad_depth": gd, "grad_albedo": ga}
    if s["kind"] == "noise":
        return {"noisy": nl.add_poisson_noise(s["tau"], s["nr_db"], s["seed"])}
    if s["kind"] == "lct":
        return {"tau": nl.lct_forward(s["params"], s["depth"], s["albedo"], s["mask"])}
    slot = s["slots"][s["turn"]]
    s["turn"] ^= 1
    if slot.busy():
        slot.event.synchronize()
    got = slot.plan(s["requests"])
    slot.launch()
    return {"tau": [g[0] for g in got], "n_active": [g[2] for g in got]}


# ---------------------------------------------------------------------------
# What a pass cannot do without

def _present(c):
    return c["px"] * c["py"] * (0.5 if c["mask"] else 1.0)


def _hist(c):
    return c["sx"] * c["sy"] * max(1, c["lx"] * c["ly"])


def _map_bytes(c):
    return c["px"] * c["py"] * (4 + (4 if c["albedo"] else 0) + (1 if c["mask"] else 0))


def _jitter_flops(c):
    r = math.ceil(2 * c["fwhm_ps"] / (2 * math.sqrt(2 * math.log(2))) / c["bin_ps"])
    return 2.0 * (2 * r + 1) * _hist(c) * c["n_bins"]


def work(case):
    c = case
    if c["kind"] == "tick":
        each = [work(r) for r in _requests(c)]
        return {k: sum(w[k] for w in each) for k in ("bytes", "flops")}
    out = 4.0 * _hist(c) * c["n_bins"]
    if c["kind"] == "noise":
        # the frame read and written; a handful of operations per element
        return {"bytes": 2 * out, "flops": 20.0 * out / 4}
    if c["kind"] == "lct":
        # the maps in, the volume out; one add per (scan point, pixel), the time resampling and the jitter
        return {"bytes": _map_bytes(c) + out, "flops": 2.0 * _hist(c) * _present(c) + _jitter_flops(c) + 3 * out}
    pairs = _hist(c) * _present(c)
    if c["kind"] == "smooth":
        # maps in, histograms out; upstream in, map gradients out; weight, arrival and two responses per pair
        return {"bytes": 2 * _map_bytes(c) + 2 * out + 8.0 * c["px"] * c["py"], "flops": 2 * 40.0 * pairs}
    # maps in, records and histograms out; 29 operations per confocal pair, 48 with separate legs, about
    # half of the pairs arriving inside the window
    return {"bytes": _map_bytes(c) + 32.0 * _present(c) + out,
            "flops": (48.0 if c["lx"] else 29.0) * 0.5 * pairs + _jitter_flops(c)}


# ---------------------------------------------------------------------------
# The same in 64 bits

def _axis64(n, half, c=0.0):
    i = torch.arange(n, dtype=torch.float64, device="cuda")
    return ((c - half) + (i + 0.5) * (2.0 * half / n)).float().double()


def _diff64(z, step, dim):
    n = z.shape[dim]
    if n < 2:
        return torch.zeros_like(z)
    lo, hi = z.narrow(dim, 0, 1), z.narrow(dim, n - 1, 1)
    first, last = (z.narrow(dim, 1, 1) - lo) / step, (hi - z.narrow(dim, n - 2, 1)) / step
    mid = (z.narrow(dim, 2, n - 2) - z.narrow(dim, 0, n - 2)) / (2 * step)
    return torch.cat([first, mid, last], dim)


def _order(c):
    """Pixel indices in record order: 16 x 16 blocks, x major, each as four stride-2 phases of 8 x 8 pixels."""
    bx, by = -(-c["px"] // 16), -(-c["py"] // 16)
    e = torch.arange(bx * by * 256, device="cuda")
    w, phase, blk = e % 64, (e // 64) % 4, e // 256
    ix = (blk // by) * 16 + (w // 8) * 2 + phase // 2
    iy = (blk % by) * 16 + (w % 8) * 2 + phase % 2
    keep = (ix < c["px"]) & (iy < c["py"])
    return ix[keep] * c["py"] + iy[keep]


def _records64(c, depth, albedo, mask):
    """x, y, z, a, n_x, n_y, n_z and pixel of the present patches, in record order."""
    z = depth.double()
    hx, hy = 2 * c["half"] / c["px"], 2 * c["half"] / c["py"]
    gx, gy = _diff64(z, hx, 0), _diff64(z, hy, 1)
    ln = torch.sqrt(1 + gx * gx + gy * gy)
    rho = albedo.double() if albedo is not None else torch.full_like(z, 0.5)
    a = rho * (hx * hy) * (ln if c["cosines"] else 1.0)
    x = _axis64(c["px"], c["half"])[:, None].expand_as(z)
    y = _axis64(c["py"], c["half"])[None, :].expand_as(z)
    here = torch.isfinite(z) & (z > 0) & (rho > 0)
    if mask is not None:
        here = here & (mask != 0)
    idx = _order(c)
    idx = idx[here.detach().reshape(-1)[idx]]
    return [t.reshape(-1)[idx] for t in (x, y, z, a, gx / ln, gy / ln, -1 / ln)] + [idx]


def _wall64(c, nx, ny):
    x = _axis64(nx, c["half"])[:, None].expand(nx, ny).reshape(-1)
    y = _axis64(ny, c["half"])[None, :].expand(nx, ny).reshape(-1)
    s = c["standoff"]
    if s <= 0:
        return x, y, torch.zeros_like(x), torch.ones_like(x)
    far = torch.sqrt((x * x + y * y) + s * s)
    return x, y, far - s, (s / far) ** 3


def _legs64(c, wall, rec):
    """Distance and weight factor of each (wall point, patch) leg."""
    x, y, z, _, nx, ny, nz, _ = rec
    dx, dy = x[None, :] - wall[0][:, None], y[None, :] - wall[1][:, None]
    r = torch.sqrt((dx * dx + dy * dy) + (z * z)[None, :])
    q = 1.0 / (r * r)
    if c["cosines"]:
        q = q * q * z[None, :] * torch.clamp(-(nx[None, :] * dx + ny[None, :] * dy + (nz * z)[None, :]), min=0.0)
    return r, q * wall[3][:, None]


def _jitter64(c, h):
    if c["fwhm_ps"] == 0:
        return h
    sig = c["fwhm_ps"] / (2 * math.sqrt(2 * math.log(2))) / c["bin_ps"]
    r, n = math.ceil(2 * sig), h.shape[1]
    tap = [math.exp(-i * i / (2 * sig * sig)) for i in range(-r, r + 1)]
    for b in range(0, h.shape[0], 65536):
        part = h[b:b + 65536]
        out = torch.zeros_like(part)
        for i in range(-r, r + 1):
            if abs(i) < n:
                to, at = (slice(i, n), slice(0, n - i)) if i >= 0 else (slice(0, n + i), slice(-i, n))
                out[:, to] += part[:, at] * (tap[i + r] / sum(tap))
        h[b:b + 65536] = out
    return h


def _simulate64(c, seed):
    depth, albedo, mask = _maps(c, seed)
    rec = _records64(c, depth, albedo, mask)
    T, inv = c["n_bins"], 1.0 / (C_LIGHT * c["bin_ps"] * 1e-12)
    det = _wall64(c, c["sx"], c["sy"])
    n_det, n = det[0].numel(), rec[0].numel()
    las = _wall64(c, c["lx"], c["ly"]) if c["lx"] else None
    n_las = las[0].numel() if las else 1
    h = torch.zeros((n_las * n_det, T), dtype=torch.float64, device="cuda")
    step = max(1, 16_000_000 // max(1, n))
    for l in range(n_las):
        if las:
            r_l, q_l = _legs64(c, [t[l:l + 1] for t in las], rec)
        for b in range(0, n_det, step):
            wall = [t[b:b + step] for t in det]
            r, q = _legs64(c, wall, rec)
            off = wall[2] + (las[2][l] if las else wall[2])
            u = (((r_l if las else r) + r) + off[:, None]) * inv
            w = (q_l if las else q) * q * rec[3][None, :]
            k = torch.floor(u).long()
            w = torch.where(k < T, w, 0.0)
            m = wall[0].numel()
            at = torch.clamp(k, max=T - 1) + (torch.arange(m, device="cuda") * T)[:, None]
            h[l * n_det + b:l * n_det + b + m].view(-1).scatter_add_(0, at.view(-1), w.view(-1))
    shape = (c["sx"], c["sy"], T) if not las else (n_las, c["sx"], c["sy"], T)
    # (the pixel index travels as the bits of a float)
    bits = rec[7].to(torch.int32).view(torch.float32).double()
    records = None if c["mask"] else torch.stack([*rec[:7], bits], 1)
    return {"tau": _jitter64(c, h).view(shape), "n_active": None, "records": records}


def _smooth64(c, seed):
    depth, albedo, mask = _maps(c, seed)
    g = _upstream(c, seed).double().view(-1, c["n_bins"])
    T, inv = c["n_bins"], 1.0 / (C_LIGHT * c["bin_ps"] * 1e-12)
    sig = c["fwhm_ps"] / (2 * math.sqrt(2 * math.log(2))) / c["bin_ps"]
    rs, norm = math.ceil(6 * sig), 1.0 / (sig * math.sqrt(2 * math.pi))
    d64, a64 = depth.double().requires_grad_(), albedo.double().requires_grad_()
    full = _records64(c, d64, a64, mask)
    rec = [t.detach().requires_grad_(i in (2, 3, 4, 5, 6)) for i, t in enumerate(full)]
    need = rec[2:7]
    grads = [torch.zeros_like(t) for t in need]
    wall_all = _wall64(c, c["sx"], c["sy"])
    S = wall_all[0].numel()
    tau = torch.zeros((S, T), dtype=torch.float64, device="cuda")
    step = max(1, 8_000_000 // max(1, rec[0].numel()))
    for b in range(0, S, step):
        wall = [t[b:b + step] for t in wall_all]
        m = wall[0].numel()
        r, q = _legs64(c, wall, rec)
        u = ((r + r) + 2 * wall[2][:, None]) * inv
        w = q * q * rec[3][None, :]
        with torch.no_grad():
            k0, ud = torch.floor(u).long(), u.detach()
            row = (torch.arange(m, device="cuda") * T)[:, None]
            g0, g1 = torch.zeros_like(ud), torch.zeros_like(ud)
            part, gpart = tau[b:b + m].view(-1), g[b:b + m].reshape(-1)
            for d in range(-rs, rs + 1):
                k = k0 + d
                x = (k.double() + 0.5) - ud
                e = torch.where((k >= 0) & (k < T), norm * torch.exp(x * x * (-0.5 / (sig * sig))), 0.0)
                at = (torch.clamp(k, 0, T - 1) + row).view(-1)
                part.scatter_add_(0, at, (w * e).view(-1))
                ge = gpart[at].view_as(e) * e
                g0 += ge
                g1 += ge * x
            g1 *= 1.0 / (sig * sig)
        for acc, new in zip(grads, torch.autograd.grad([w, u], need, [g0, w.detach() * g1], allow_unused=True)):
            if new is not None:
                acc += new
    gd, ga = torch.autograd.grad(full[2:7], [d64, a64], grads, allow_unused=True)
    return {"tau": tau.view(c["sx"], c["sy"], T), "grad_depth": gd, "grad_albedo": ga}


def _lct64(c, seed):
    depth, albedo, mask = _maps(c, seed)
    n, m = c["sx"], c["n_bins"]
    dt = c["bin_ps"] * 1e-12
    dz, slope = C_LIGHT * dt / 2, c["half"] / (m * C_LIGHT * dt)
    z = depth.double().view(-1)
    rho = albedo.double().view(-1)
    j = torch.floor(z / dz)
    ok = torch.isfinite(z) & (z > 0) & (rho > 0) & (j < m)
    if mask is not None:
        ok &= mask.view(-1) != 0
    at = torch.nonzero(ok)[:, 0]
    big = j[at].long() + 1
    layer, amp = (big * big - 1) // m, rho[at] / big.double() / m
    # the cone's layer of each lateral offset: the nearest to (4 slope)^2 (x^2 + y^2), both at a tie
    o = torch.arange(n, dtype=torch.float64, device="cuda") / n
    zs = (4.0 * slope) ** 2 * ((o * o)[:, None] + (o * o)[None, :]) * m
    lo = torch.floor(zs)
    frac = zs - lo
    k1 = torch.where(frac <= 0.5, lo, lo + 1).clamp(max=4.0 * m).long()
    k2 = torch.where(frac == 0.5, lo + 1, torch.full_like(lo, 4.0 * m)).clamp(max=4.0 * m).long()
    conv = torch.zeros((n * n, m), dtype=torch.float64, device="cuda")
    px, py = at // n, at % n
    s = torch.arange(n * n, device="cuda")
    step = max(1, 16_000_000 // max(1, at.numel()))
    for b in range(0, n * n, step):
        p = s[b:b + step]
        dx, dy = ((p // n)[:, None] - px[None, :]).abs(), ((p % n)[:, None] - py[None, :]).abs()
        for tab in ([k1, k2] if bool((k2 < m).any()) else [k1]):
            k = tab[dx, dy] + layer[None, :]
            w = torch.where(k < m, amp[None, :], 0.0)
            idx = torch.clamp(k, max=m - 1) + (torch.arange(p.numel(), device="cuda") * m)[:, None]
            conv[b:b + step].view(-1).scatter_add_(0, idx.view(-1), w.reshape(-1))
    # bin j: the mean over the fine samples [j^2, (j + 1)^2) of the coarse ones of m each, over (J dz)^3
    jj = torch.arange(m, device="cuda")
    lo, hi = jj * jj, (jj + 1) * (jj + 1)
    cs = torch.arange(m, device="cuda")
    ov = (torch.minimum(hi[:, None], (cs[None, :] + 1) * m) - torch.maximum(lo[:, None], cs[None, :] * m)).clamp(min=0)
    rt = ov.double() / (2 * jj + 1).double()[:, None] / (((jj + 1).double() * dz) ** 3)[:, None]
    return {"tau": _jitter64(c, conv @ rt.t().contiguous()).view(n, n, m)}


def exact(case, seed):
    c = case
    if c["kind"] == "noise":
        return None   # random counts by a fixed recipe: whole numbers over one scale, the same or wrong
    if c["kind"] == "tick":
        each = [_simulate64(r, seed * 1000 + i)["tau"] for i, r in enumerate(_requests(c))]
        return {"tau": each, "n_active": [None] * len(each)}
    return {"simulate": _simulate64, "smooth": _smooth64, "lct": _lct64}[c["kind"]](c, seed)
