"""The workloads that performance is measured on: reconstruction of event
batches from their hits, the find with its refits, fitting, seeding from the
hits, and the propagation surrogate's training, through the package's binding.

Every case is a dict of plain values; `prepare` makes its inputs on the GPU from
a seed (particles in a solenoid crossing a layered detector: scattering, lost
hits and noise, as the synthetic events of the tests), `run` takes one pass and
`work` states the bytes and operations the pass cannot do without.  `exact`
gives the Kalman fit in 64 bits.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1811_04141_amd import mkf

KAPPA = 0.299792458e-2                 # GeV / (T cm)
BZ = 3.8                               # T
BARREL_R = (4.0, 7.0, 11.0, 16.0, 25.0, 34.0, 43.0, 52.0, 61.0, 70.0)
DISK_Z = tuple(120.0 + 20.0 * i for i in range(9))
SIGMA_U, SIGMA_V = 0.003, 0.01         # cm: r-phi; z (barrel) or r (disk)
MS_SIGMA = 0.001                       # rad per crossed layer
STEREO, SIGMA_PERP = 0.1, 1.5          # rad, cm
LOSS, NOISE = 0.02, 0.3
# solenoid-like field: Bz = b0 (1 + c_r2 r^2 + c_z2 z^2 + c_z4 z^4)
FIELD = SimpleNamespace(b0=3.8, c_r2=-1e-6, c_z2=-4.9e-6, c_z4=-1.1e-11, h_max=5.0)
SEEDING = SimpleNamespace(layers=(0, 1, 2), pt_min=0.25, d0_max=0.1, z0_max=20.0, dz_max=0.1)
CLEANING = SimpleNamespace(tol_ipt=0.1, tol_eta=0.02, tol_phi=0.02)
TRACK_FIELDS = ("seed_id", "status", "n_hits", "n_miss", "plan_len", "chi2", "par", "cov",
                "plan", "hit")
TRAIN_LOSS_W = (1.0, 0.01, 0.01, 0.01, 0.01, 0.01, 0.01)


def listed():
    base = dict(detector="barrel_endcap", events=1, tracks=200, spread=0.0, form="batched",
                n_cand=6, material=False, field=False)

    def case(name, path, **kw):
        return dict(base, name=name, path=path, **kw)

    return [
        # One small event, hits to tracks: the least a program can ask for, where
        # the calls' own latency counts.
        case("event_barrel_200", "reconstruct", detector="barrel"),
        # One ordinary event (pile-up, noise), hits to tracks: event-by-event use.
        case("event_5000", "reconstruct", tracks=5000),
        # A batch of events at once, hits to tracks: throughput use, the repository's
        # realistic workload.
        case("batch_100x5000", "reconstruct", events=100, tracks=5000),
        # The find and the refit towards the vertex of loaded events: the hot path on
        # the realistic workload, with the launch shape the autotuner keeps for it.
        case("find_refit_100x5000", "refit", events=100, tracks=5000),
        # The same in the learned-surrogate form, replayed as a graph, on uneven events:
        # the benchmark's form.
        case("find_surrogate_uneven", "refit", events=37, tracks=3000, spread=1.0,
             form="surrogate"),
        # Material map and parameterised field together.
        case("find_extended_20x2000", "refit", events=20, tracks=2000, material=True, field=True),
        # Layer-synchronous find (the default form) and smoothing, on the geometry with
        # stereo layers and holes.
        case("find_smooth_stereo", "smooth", detector="stereo", events=10, tracks=2000,
             form="layers"),
        # Seeds from the hits alone.
        case("triplets_20x5000", "triplets", events=20, tracks=5000),
        # From triplet seeds to tracks without duplicates.
        case("triplet_tracks_4x5000", "triplet_tracks", events=4, tracks=5000),
        # Fit of many tracks with known hits: 26 layers each (the fit stress workload).
        dict(name="fit_1M_26", path="fit", tracks=1000000, steps=26, ragged=False),
        # A few tracks, of uneven length: one event's refit.
        dict(name="fit_1003_13", path="fit", tracks=1003, steps=13, ragged=True),
        # Training of the surrogate and its inference on held-out samples.
        dict(name="surrogate_train", path="train", samples=131072, epochs=2, batch=512,
             infer=100003),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(["reconstruct", "reconstruct", "reconstruct", "refit", "refit", "smooth",
                       "triplets", "triplet_tracks", "fit", "fit", "train"])
    if path == "fit":
        steps = rng.randint(5, 30)
        return dict(path="fit", tracks=size(500, 20000000 // steps), steps=steps,
                    ragged=rng.random() < 0.5)
    if path == "train":
        batch = rng.choice([128, 256, 512, 1024])
        return dict(path="train", samples=batch * rng.randint(20, 400), epochs=rng.randint(1, 2),
                    batch=batch, infer=size(1000, 1000000))
    most = {"reconstruct": 400000, "refit": 400000, "smooth": 60000, "triplets": 100000,
            "triplet_tracks": 20000}[path]
    tracks = size(50, 6000)
    events = max(1, min(size(1, 100), most // (2 * tracks)))
    detector = rng.choice(["barrel_endcap", "barrel_endcap", "stereo", "barrel"])
    field = path in ("reconstruct", "refit") and rng.random() < 0.2
    forms = {"smooth": ["layers", "batched"], "refit": ["batched", "layers", "surrogate"]}
    return dict(path=path, detector=detector, events=events, tracks=tracks,
                spread=round(rng.uniform(0.1, 0.7), 2) if events > 1 and rng.random() < 0.5 else 0.0,
                form=rng.choice(forms.get(path, ["batched", "batched", "layers"])),
                n_cand=rng.choice([6, 6, 6, 4, 8]), material=rng.random() < 0.2, field=field)


# ------------------------------------------------------------------ inputs


def detector_layers(detector):
    """Layer records: 10 cylinders, then 9 disks on each side unless barrel only."""
    vu, vv = SIGMA_U ** 2, SIGMA_V ** 2

    def layer(kind, pos, lo, hi, **kw):
        return SimpleNamespace(**dict(dict(
            kind=kind, pos=pos, ext_lo=lo, ext_hi=hi, var_u_max=vu, var_v_max=vv, n_phi_bins=256,
            n_q_bins=16, stereo=0.0, hole_lo=0.0, hole_hi=0.0), **kw))

    out = [layer(0, r, -100.0, 100.0) for r in BARREL_R]
    if detector != "barrel":
        out += [layer(1, z, 20.0, 110.0) for z in DISK_Z]
        out += [layer(1, -z, 20.0, 110.0) for z in DISK_Z]
    if detector == "stereo":
        c2, s2 = math.cos(STEREO) ** 2, math.sin(STEREO) ** 2
        vp = SIGMA_PERP ** 2
        for k in (4, 6):
            out[k].stereo = STEREO
            out[k].var_u_max, out[k].var_v_max = c2 * vu + s2 * vp, s2 * vu + c2 * vp
        out[5].hole_lo, out[5].hole_hi = -2.0, 2.0
        for d in out[10:]:
            d.hole_lo, d.hole_hi = 50.0, 55.0
    return out


def find_config(case):
    return SimpleNamespace(
        bz=BZ, kappa=KAPPA, chi2_cut=30.0, n_cand=case.get("n_cand", 6), max_holes=3,
        ms_sigma=0.0 if case.get("detector") == "barrel" else MS_SIGMA, edge_margin=2.0,
        l_min=1e-4, init_var=(1.0, 1.0, 1.0, 1.0, 0.01, 0.01))


def material_map():
    """1.5% of a radiation length and 0.1 g/cm^2 per layer, half as much again
    beyond |z| = 50 cm."""
    n_r, n_z, z_max = 24, 30, 300.0
    z = -z_max + (np.arange(n_z) + 0.5) * (2.0 * z_max / n_z)
    f = np.where(np.abs(z) > 50.0, 1.5, 1.0)[:, None] * np.ones((1, n_r))
    return SimpleNamespace(n_r=n_r, n_z=n_z, r_max=120.0, z_max=z_max, mass=0.13957, k_max=10.0,
                           x_x0=(0.015 * f).astype(np.float32), xi=(0.1 * f).astype(np.float32))


class Rng:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def uniform(self, n, lo=0.0, hi=1.0):
        return torch.rand(n, generator=self.g, device="cuda", dtype=torch.float64) * (hi - lo) + lo

    def normal(self, n, sigma=1.0):
        return torch.randn(n, generator=self.g, device="cuda", dtype=torch.float64) * sigma


def bz_at(field, x, y, z):
    if not field:
        return torch.full_like(x, BZ)
    r2, z2 = x * x + y * y, z * z
    return FIELD.b0 * (1.0 + FIELD.c_r2 * r2 + FIELD.c_z2 * z2 + FIELD.c_z4 * z2 * z2)


def path_to(x, y, z, phi, theta, omega, kind, pos):
    """Transverse path of an outgoing helix to a cylinder (from inside) or a
    plane z = pos (NaN where there is none within half a turn)."""
    if kind == 0:
        a = x * torch.cos(phi) + y * torch.sin(phi)
        c = y * torch.cos(phi) - x * torch.sin(phi)
        g0 = x * x + y * y - pos * pos
        alpha = 1.0 + c * omega + 0.25 * g0 * omega * omega
        tau = -g0 / (a + torch.sqrt(a * a - alpha * g0))
        l = 2.0 / omega * torch.atan(0.5 * omega * tau)
    else:
        l = (pos - z) * torch.tan(theta)
    return torch.where((l > 1e-4) & (torch.abs(omega) * l < math.pi), l, torch.nan)


def advance(x, y, z, phi, theta, omega, l):
    h = 0.5 * omega * l
    chord = l * torch.sinc(h / math.pi)
    return (x + chord * torch.cos(phi + h), y + chord * torch.sin(phi + h),
            z + l / torch.tan(theta), phi + omega * l)


def make_events(case, seed):
    """Hits of all events in random order within each, and the triplet of every
    particle's first three hits."""
    rng = Rng(seed)
    layers = detector_layers(case["detector"])
    clean = case["detector"] == "barrel"
    n_ev = case["events"]
    # uneven events: sizes spread over e^-spread .. e^spread, in random order
    size = torch.linspace(-case["spread"], case["spread"], n_ev, dtype=torch.float64, device="cuda")
    count = torch.round(case["tracks"] * torch.exp(size)).long()[torch.argsort(rng.uniform(n_ev))]
    ev = torch.repeat_interleave(torch.arange(n_ev, device="cuda"), count)
    n = ev.numel()
    pt = torch.exp(rng.uniform(n, math.log(0.5 if clean else 0.3), math.log(10.0)))
    eta = rng.uniform(n, -0.8, 0.8) if clean else rng.uniform(n, -2.4, 2.4)
    charge = torch.where(rng.uniform(n) < 0.5, -1.0, 1.0)
    phi, theta = rng.uniform(n, -math.pi, math.pi), 2.0 * torch.atan(torch.exp(-eta))
    x, y, z = rng.normal(n, 0.01), rng.normal(n, 0.01), rng.normal(n, 5.0)
    turned = torch.zeros_like(x)
    side = torch.where(theta < 0.5 * math.pi, 1.0, -1.0)
    xs, ys, zs, ids, seen = [], [], [], [], []
    surfaces = list(range(10)) + ([] if clean else list(range(10, 19)))
    for k in surfaces:
        L = layers[k]
        pos = L.pos if L.kind == 0 else L.pos * side
        omega = -KAPPA * bz_at(case["field"], x, y, z) * charge / pt
        l = path_to(x, y, z, phi, theta, omega, L.kind, pos)
        if case["field"]:  # the field half-way
            x1, y1, z1, _ = advance(x, y, z, phi, theta, omega, l)
            mid = bz_at(True, 0.5 * (x + x1), 0.5 * (y + y1), 0.5 * (z + z1))
            omega = torch.where(torch.isfinite(mid), -KAPPA * mid * charge / pt, omega)
            l = path_to(x, y, z, phi, theta, omega, L.kind, pos)
        x1, y1, z1, phi1 = advance(x, y, z, phi, theta, omega, l)
        q = z1 if L.kind == 0 else torch.hypot(x1, y1)
        on = (q >= L.ext_lo) & (q <= L.ext_hi) & (turned + torch.abs(omega) * l < math.pi)
        x, y, z = torch.where(on, x1, x), torch.where(on, y1, y), torch.where(on, z1, z)
        phi = torch.where(on, phi1, phi)
        turned = torch.where(on, turned + torch.abs(omega) * l, turned)
        # the smeared hit, on the surface
        du, dv = rng.normal(n, SIGMA_U), rng.normal(n, SIGMA_V)
        if L.stereo:
            c, s, dp = math.cos(L.stereo), math.sin(L.stereo), rng.normal(n, SIGMA_PERP)
            du, dv = c * du - s * dp, s * du + c * dp
        r = torch.full_like(x, L.pos) if L.kind == 0 else torch.hypot(x, y) + dv
        ph = torch.atan2(y, x) + du / (L.pos if L.kind == 0 else torch.hypot(x, y))
        xs.append(r * torch.cos(ph))
        ys.append(r * torch.sin(ph))
        zs.append(z + dv if L.kind == 0 else pos + torch.zeros_like(z))
        ids.append(torch.full_like(ev, k) if L.kind == 0 else torch.where(side > 0, k, k + 9))
        hole = (q > L.hole_lo) & (q < L.hole_hi) if L.hole_lo < L.hole_hi else torch.zeros_like(on)
        seen.append(on & ~hole & (rng.uniform(n) >= (0.0 if clean else LOSS)))
        if not clean:  # scattering, |p| kept
            p_tot = pt / torch.sin(theta)
            phi = torch.where(on, phi + rng.normal(n, MS_SIGMA) / torch.sin(theta), phi)
            theta = torch.where(on, theta + rng.normal(n, MS_SIGMA), theta)
            pt = p_tot * torch.sin(theta)
    seen = torch.stack(seen, 1)
    x, y, z, lay = (torch.stack(v, 1)[seen] for v in (xs, ys, zs, ids))
    trk = torch.arange(n, device="cuda")[:, None].expand(n, len(surfaces))[seen]
    hev, n_true = ev[trk], trk.numel()
    if not clean:  # noise: a share of each layer's hits, uniform over it
        nl = len(layers)
        per = torch.bincount(hev * nl + lay, minlength=n_ev * nl)
        cell = torch.repeat_interleave(torch.arange(n_ev * nl, device="cuda"),
                                       torch.round(per * NOISE).long())
        m = cell.numel()
        tab = {f: torch.tensor([float(getattr(L, f)) for L in layers], dtype=torch.float64,
                               device="cuda")[cell % nl]
               for f in ("kind", "pos", "ext_lo", "ext_hi", "hole_lo", "hole_hi")}
        u, ph = rng.uniform(m), rng.uniform(m, -math.pi, math.pi)
        bar = tab["kind"] == 0
        zn = torch.where(bar, tab["ext_lo"] + u * (tab["ext_hi"] - tab["ext_lo"]), tab["pos"])
        rn = torch.where(bar, tab["pos"],
                         torch.sqrt(tab["ext_lo"] ** 2 + u * (tab["ext_hi"] ** 2 - tab["ext_lo"] ** 2)))
        q = torch.where(bar, zn, rn)
        keep = ~((q > tab["hole_lo"]) & (q < tab["hole_hi"]))
        x = torch.cat([x, (rn * torch.cos(ph))[keep]])
        y = torch.cat([y, (rn * torch.sin(ph))[keep]])
        z = torch.cat([z, zn[keep]])
        lay = torch.cat([lay, (cell % nl)[keep]])
        hev = torch.cat([hev, (cell // nl)[keep]])
    # random order within each event
    order = torch.argsort(hev + rng.uniform(hev.numel()))
    place = torch.empty_like(order)
    place[order] = torch.arange(order.numel(), device="cuda")
    off = torch.zeros(n_ev + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(torch.bincount(hev, minlength=n_ev), 0)
    vv = torch.full_like(x, SIGMA_V ** 2)
    for k, L in enumerate(layers):
        if L.stereo:
            vv[lay == k] = SIGMA_PERP ** 2
    hits = [v[order].float() for v in (x, y, z)]
    hits += [torch.full_like(hits[0], SIGMA_U ** 2), vv[order].float(), lay[order].int()]
    # seeds: the first three hits of each particle (true hits come track by track);
    # in place of the few particles with fewer hits, others' seeds a second time
    local = (place - off[hev])[:n_true].int()
    n_hits = torch.bincount(trk, minlength=n)
    first = torch.cumsum(n_hits, 0) - n_hits
    full = (n_hits >= 3).nonzero()[:, 0]
    full = full[torch.arange(n, device="cuda") % full.numel()]
    at = first[full]
    seed_hits = torch.stack([local[at], local[at + 1], local[at + 2]], 1).contiguous()
    return SimpleNamespace(layers=layers, ev_off=off.cpu().numpy(), hits=hits,
                           seed_event=ev[full].int(), seed_hits=seed_hits)


def make_context(case, ev):
    flags = {"layers": 0, "batched": mkf.F_BATCHED,
             "surrogate": mkf.F_BATCHED | mkf.F_SURROGATE | mkf.F_GRAPH}[case["form"]]
    # graph replay wants a stream of its own
    stream = torch.cuda.Stream() if flags & mkf.F_GRAPH else None
    ctx = mkf.Context(find_config(case), flags=flags, stream=stream.cuda_stream if stream else None)
    ctx.load_geometry(ev.layers)
    if case["material"]:
        ctx.load_material(material_map())
    if case["field"]:
        ctx.load_field(FIELD)
    torch.cuda.synchronize()
    if flags & mkf.F_SURROGATE:
        ctx.surrogate_train(1 << 18, 1, 512, 3e-3, 11, TRAIN_LOSS_W)
    return ctx, stream


def triplet_capacity(case):
    return int(case["events"] * case["tracks"] * (4 + 1e-6 * case["tracks"] ** 2)) + 4096


def make_triplets(s):
    """The hits' triplet seeds as sorted keys, event and three hits (the library's
    order within one bin of its index is not fixed)."""
    n = s.ctx.make_seeds(SEEDING, s.tr_event.numel(), s.tr_event, s.tr_hits)
    key = s.tr_event[:n].long()
    for k in range(3):
        key = (key << 18) | s.tr_hits[:n, k]
    s.tr_key[:n] = torch.sort(key).values
    return n


def prepare(case, seed):
    if case["path"] == "fit":
        return prepare_fit(case, seed)
    if case["path"] == "train":
        return prepare_train(case, seed)
    ev = make_events(case, seed)
    ctx, stream = make_context(case, ev)
    s = SimpleNamespace(case=case, ev=ev, ctx=ctx, stream=stream, n=ev.seed_event.numel())
    if case["path"] == "reconstruct":
        return s
    if case["path"] in ("refit", "smooth") and case["form"] != "layers":
        ctx.set_tuning(3, 3)
    ctx.load_hits(ev.ev_off, *ev.hits)
    if case["path"] in ("triplets", "triplet_tracks"):
        cap = triplet_capacity(case)
        s.tr_event = torch.empty(cap, dtype=torch.int32, device="cuda")
        s.tr_hits = torch.empty((cap, 3), dtype=torch.int32, device="cuda")
        s.tr_key = torch.full((cap,), -1, dtype=torch.int64, device="cuda")
    if case["path"] == "triplet_tracks":
        key = s.tr_key[:make_triplets(s)]
        mask = (1 << 18) - 1
        ev.seed_event = (key >> 54).int().contiguous()
        ev.seed_hits = torch.stack([(key >> 36) & mask, (key >> 18) & mask, key & mask], 1)
        ev.seed_hits = ev.seed_hits.int().contiguous()
        s.n = ev.seed_event.numel()
        # buffers for as many seeds as events of this size may give
        s.keep = torch.zeros(cap, dtype=torch.int32, device="cuda")
        s.dup = torch.zeros(cap, dtype=torch.int32, device="cuda")
    elif case["path"] in ("refit", "smooth"):
        ctx.seed(ev.seed_event, ev.seed_hits)
        rows = (s.n,) if case["path"] == "refit" else (s.n, mkf.MAX_PLAN + 1)
        s.par = torch.zeros(rows + (6,), device="cuda")
        s.cov = torch.zeros(rows + (21,), device="cuda")
        s.chi2 = torch.zeros(s.n, device="cuda")
        s.status = torch.zeros(s.n, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
    return s


def prepare_train(case, seed):
    ctx = mkf.Context(find_config(case))
    ctx.load_geometry(detector_layers("barrel"))
    n = case["infer"]
    x, t = torch.empty((n, 8), device="cuda"), torch.empty((n, 7), device="cuda")
    valid = torch.empty(n, device="cuda")
    ctx.surrogate_samples(n, seed + 1, x, t, valid)
    return SimpleNamespace(case=case, ctx=ctx, seed=seed, start=ctx.surrogate_get(), x=x,
                           y=torch.zeros((n, 7), device="cuda"))


def prepare_fit(case, seed):
    """Half the tracks in cylinders, half in disks of either side; the fit starts
    at the vertex, displaced by a draw of its own prior."""
    rng = Rng(seed)
    n, m = case["tracks"], case["steps"]
    radii = torch.sort(rng.uniform(m, 4.0, 100.0)).values
    planes = torch.sort(rng.uniform(m, 40.0, 320.0)).values
    disk = rng.uniform(n) < 0.5
    side = torch.where(rng.uniform(n) < 0.5, -1.0, 1.0)
    eta = torch.where(disk, side * rng.uniform(n, 1.8, 2.4), rng.uniform(n, -1.0, 1.0))
    pt = torch.exp(rng.uniform(n, 0.0, math.log(10.0)))
    ipt = torch.where(rng.uniform(n) < 0.5, -1.0, 1.0) / pt
    phi0, theta = rng.uniform(n, -math.pi, math.pi), 2.0 * torch.atan(torch.exp(-eta))
    x, y, z, phi = rng.normal(n, 0.005), rng.normal(n, 0.005), rng.normal(n, 1.0), phi0
    init = torch.stack([x, y, z, ipt, phi0, theta], 1)
    sigma = torch.tensor([0.01, 0.01, 0.1, 0.05, 1e-3, 1e-3], dtype=torch.float64, device="cuda")
    sigma = sigma.repeat(n, 1)
    sigma[:, 3] *= ipt.abs()
    init = init + rng.normal((n, 6)) * sigma
    cov = torch.zeros((n, 21), dtype=torch.float64, device="cuda")
    cov[:, [0, 6, 11, 15, 18, 20]] = sigma ** 2
    omega = -KAPPA * BZ * ipt
    s = SimpleNamespace(case=case, n=n)
    s.kind = disk.to(torch.int8).repeat(m, 1)
    cols = {k: torch.empty((m, n), device="cuda") for k in ("pos", "x", "y", "z")}
    for k in range(m):
        pos = torch.where(disk, planes[k] * side, radii[k])
        l = torch.where(disk, path_to(x, y, z, phi, theta, omega, 1, pos),
                        path_to(x, y, z, phi, theta, omega, 0, pos))
        x, y, z, phi = advance(x, y, z, phi, theta, omega, l)
        du, dv = rng.normal(n, SIGMA_U), rng.normal(n, SIGMA_V)
        r = torch.where(disk, torch.hypot(x, y) + dv, pos)
        ph = torch.atan2(y, x) + du / torch.hypot(x, y)
        for f, v in (("pos", pos), ("x", r * torch.cos(ph)), ("y", r * torch.sin(ph)),
                     ("z", torch.where(disk, pos, z + dv))):
            cols[f][k] = v.float()
    s.hits = [cols[f] for f in ("pos", "x", "y", "z")]
    s.hits += [torch.full((m, n), v ** 2, device="cuda") for v in (SIGMA_U, SIGMA_V)]
    length = torch.full((n,), m, device="cuda", dtype=torch.int64)
    if case["ragged"]:
        length = (rng.uniform(n, 0.5, 1.0) * (m + 1)).long().clamp(1, m)
    s.len = length.int()
    s.par, s.cov = init.float().contiguous(), cov.float().contiguous()
    s.out = [torch.zeros((n, 6), device="cuda"), torch.zeros((n, 21), device="cuda"),
             torch.zeros(n, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")]
    s.ctx = mkf.Context(find_config(case))
    return s


# --------------------------------------------------------------------- run


def run(s):
    path, ctx = s.case["path"], s.ctx
    if path == "fit":
        ctx.fit(s.kind, *s.hits, s.len, s.par, s.cov, *s.out)
        return s.out
    if path == "train":
        c = s.case
        ctx.surrogate_set(s.start)
        rep = ctx.surrogate_train(c["samples"], c["epochs"], c["batch"], 3e-3, s.seed, TRAIN_LOSS_W)
        ctx.surrogate_infer(s.x, s.y)
        return {"weights": ctx.surrogate_get(), "y": s.y, "loss_first": rep["loss_first"],
                "loss_last": rep["loss_last"], "n_valid": rep["n_valid"]}
    if path == "triplets":
        return {"n": make_triplets(s), "key": s.tr_key}
    if path == "reconstruct":
        ctx.load_hits(s.ev.ev_off, *s.ev.hits)
        ctx.seed(s.ev.seed_event, s.ev.seed_hits)
        ctx.find()
        tracks = ctx.get_tracks(s.n)
        return {f: tracks[f] for f in TRACK_FIELDS}
    if path == "triplet_tracks":
        ctx.seed(s.ev.seed_event, s.ev.seed_hits)
        ctx.clean_seeds(CLEANING, s.keep)
        kept = s.keep[:s.n].nonzero()[:, 0]
        ctx.seed(s.ev.seed_event[kept], s.ev.seed_hits[kept])
        ctx.find()
        n_dup = ctx.find_duplicates(0.5, s.dup)
        tracks = ctx.get_tracks(s.keep.numel())
        return {"keep": s.keep, "duplicate": s.dup, "n_dup": n_dup,
                "tracks": {f: tracks[f] for f in TRACK_FIELDS}}
    ctx.find()
    if path == "refit":
        ctx.backward_fit(s.par, s.cov, s.chi2, s.status)
        return {"par": s.par, "cov": s.cov, "chi2": s.chi2, "status": s.status}
    ctx.smooth(s.par, s.cov, s.status)
    return {"par": s.par, "cov": s.cov, "n": s.status}


# -------------------------------------------------------------------- work


def work(case):
    """Each input once and each output once; operations counted with a
    transcendental as one (780 per candidate and layer, 727 per fitted hit)."""
    path = case["path"]
    if path == "fit":
        n, m = case["tracks"], case["steps"] * (0.75 if case["ragged"] else 1.0)
        return {"bytes": n * (25.0 * m + 4 + 108 + 108 + 8), "flops": 727.0 * n * m}
    if path == "train":
        n = case["samples"] * case["epochs"]
        return {"bytes": 60.0 * n + 60.0 * case["infer"],
                "flops": 29312.0 * n + 10112.0 * case["infer"]}
    n = float(case["events"] * case["tracks"]) * (1.0 + case["spread"] ** 2 / 6.0)
    barrel = case["detector"] == "barrel"
    hits = n * (10.0 if barrel else 15.2)            # with noise
    find = 780.0 * n * (8.0 if barrel else 43.0)     # candidate-layer steps
    on_track = 10.0 if barrel else 11.6
    if path == "reconstruct":
        return {"bytes": 24.0 * hits + n * (16 + 288), "flops": find}
    if path == "refit":
        return {"bytes": 32.0 * hits + n * (112 + 32 + 116), "flops": find + 727.0 * n * on_track}
    if path == "smooth":
        return {"bytes": 32.0 * hits + n * (112 + 32 + 108 * on_track),
                "flops": find + 3 * 727.0 * n * on_track}
    triplets = n * (1.0 if barrel else 1.0 + 1.6e-7 * case["tracks"] ** 2)
    if path == "triplets":
        return {"bytes": 32.0 * n * 3.9 + 16.0 * triplets, "flops": 400.0 * triplets}
    return {"bytes": 32.0 * hits + triplets * (16 + 4 + 288 + 4),
            "flops": 780.0 * triplets * (8.0 if barrel else 43.0)}


# ------------------------------------------------------------------- exact


def exact(case, seed):
    """The Kalman fit in 64 bits (the other paths choose among hits, which has
    no value of more bits)."""
    if case["path"] != "fit":
        return None
    s = prepare_fit(case, seed)
    s.ctx.close()
    parts = [fit_exact(s, lo, min(lo + 250000, s.n)) for lo in range(0, s.n, 250000)]
    return [torch.cat([p[k] for p in parts]) for k in range(3)] + [None]


def fit_exact(s, lo, hi):
    f64 = torch.float64
    n = hi - lo
    iu = torch.triu_indices(6, 6, device="cuda")
    p = s.par[lo:hi].to(f64)
    C = torch.zeros((n, 6, 6), dtype=f64, device="cuda")
    C[:, iu[0], iu[1]] = s.cov[lo:hi].to(f64)
    C[:, iu[1], iu[0]] = s.cov[lo:hi].to(f64)
    chi2 = torch.zeros(n, dtype=f64, device="cuda")
    alive = torch.ones(n, dtype=torch.bool, device="cuda")
    # settings as the single-precision numbers the library is given
    mkb = -float(np.float32(np.float32(KAPPA) * np.float32(BZ)))
    ms2 = float(np.float32(MS_SIGMA)) ** 2
    eye = torch.eye(6, dtype=f64, device="cuda")
    for k in range(s.kind.shape[0]):
        disk = s.kind[k, lo:hi] == 1
        pos, hx, hy, hz, vu, vv = (v[k, lo:hi].to(f64) for v in s.hits)
        x, y, z, ipt, phi, theta = p.unbind(1)
        w = mkb * ipt
        l = torch.where(disk, path_to(x, y, z, phi, theta, w, 1, pos),
                        path_to(x, y, z, phi, theta, w, 0, pos))
        alive = alive & (k < s.len[lo:hi]) & torch.isfinite(l)
        l = torch.where(torch.isfinite(l), l, 1.0)
        x1, y1, z1, phi1 = advance(x, y, z, phi, theta, w, l)
        # Jacobian at fixed path, then the constraint to the surface
        h = 0.5 * w * l
        sn, ch = torch.sin(h), torch.cos(h)
        small = h.abs() < 1e-3
        hs = torch.where(small, 1.0, h)
        sinc = torch.where(small, 1.0 - h * h / 6.0, sn / hs)
        dsinc = torch.where(small, -h / 3.0 + h ** 3 / 30.0, (hs * ch - sn) / (hs * hs))
        cp, sp = torch.cos(phi + h), torch.sin(phi + h)
        D = eye.repeat(n, 1, 1)
        half = 0.5 * l * mkb
        D[:, 0, 3] = l * half * (dsinc * cp - sinc * sp)
        D[:, 0, 4] = -l * sinc * sp
        D[:, 1, 3] = l * half * (dsinc * sp + sinc * cp)
        D[:, 1, 4] = l * sinc * cp
        D[:, 2, 5] = -l / torch.sin(theta) ** 2
        D[:, 4, 3] = l * mkb
        zero = torch.zeros_like(x)
        t = torch.stack([torch.cos(phi1), torch.sin(phi1), 1.0 / torch.tan(theta), zero, w, zero], 1)
        nv = torch.stack([torch.where(disk, 0.0, x1), torch.where(disk, 0.0, y1),
                          torch.where(disk, 1.0, 0.0).to(f64), zero, zero, zero], 1)
        P = eye - t[:, :, None] * nv[:, None, :] / (nv * t).sum(1)[:, None, None]
        F = torch.bmm(P, D)
        C1 = torch.bmm(torch.bmm(F, C), F.transpose(1, 2).contiguous())
        sth, a = torch.sin(theta), ipt / torch.tan(theta)
        C1[:, 3, 3] += a * a * ms2
        C1[:, 3, 5] -= a * ms2
        C1[:, 5, 3] -= a * ms2
        C1[:, 4, 4] += ms2 / (sth * sth)
        C1[:, 5, 5] += ms2
        # residual along the azimuth and along z (cylinder) or r (disk)
        r = torch.hypot(x1, y1)
        H = torch.zeros((n, 2, 6), dtype=f64, device="cuda")
        H[:, 0, 0], H[:, 0, 1] = -y1 / r, x1 / r
        H[:, 1, 0], H[:, 1, 1] = torch.where(disk, x1 / r, 0.0), torch.where(disk, y1 / r, 0.0)
        H[:, 1, 2] = torch.where(disk, 0.0, 1.0).to(f64)
        alive = alive & (disk | (x1 * hx + y1 * hy > 0.0))
        res = torch.bmm(H, torch.stack([hx - x1, hy - y1, hz - z1, zero, zero, zero], 1)[:, :, None])
        CH = torch.bmm(C1, H.transpose(1, 2).contiguous())
        S = torch.bmm(H, CH) + torch.diag_embed(torch.stack([vu, vv], 1))
        det = S[:, 0, 0] * S[:, 1, 1] - S[:, 0, 1] * S[:, 1, 0]
        Si = torch.stack([S[:, 1, 1], -S[:, 0, 1], -S[:, 1, 0], S[:, 0, 0]], 1).view(n, 2, 2)
        Si = Si / det[:, None, None]
        K = torch.bmm(CH, Si)
        q = torch.stack([x1, y1, z1, ipt, phi1, theta], 1) + torch.bmm(K, res)[:, :, 0]
        q[:, 4] = torch.remainder(q[:, 4] + math.pi, 2.0 * math.pi) - math.pi
        J = eye - torch.bmm(K, H)
        V = torch.diag_embed(torch.stack([vu, vv], 1))
        C2 = torch.bmm(torch.bmm(J, C1), J.transpose(1, 2).contiguous())
        C2 = C2 + torch.bmm(torch.bmm(K, V), K.transpose(1, 2).contiguous())
        add = torch.bmm(torch.bmm(res.transpose(1, 2).contiguous(), Si), res)[:, 0, 0]
        chi2 = torch.where(alive, chi2 + add, chi2)
        p = torch.where(alive[:, None], q, p)
        C = torch.where(alive[:, None, None], C2, C)
    return p, C[:, iu[0], iu[1]], chi2
