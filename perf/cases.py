"""The work that programs have this library do, as cases that can be timed.

Every case goes through the public entry points of paper_1204_5041_amd: maps
of boxes of string segments in both arithmetic forms, maps of batches of
boxes under visibility rules, a differentiation step, Eq. (1) at chosen
directions, stacked healpix-cone boxes, flat-sky patches, power spectra and
light-cone event recording.  Segments follow the recipe of `synth`, drawn on
the GPU.  `listed` names the cases, `draw` gives more of the same ranges,
`prepare` makes what a program holds before the call, `run` is one pass,
`work` the bytes and operations a pass cannot do without, and `exact` the
pass's outputs in 64 bits from plain torch.

Maps of the FP32C form and flat-sky maps come from FP32 arithmetic (3e-7 of
the map's rms) and are handed on in single precision, which is also how the
differentiable map returns the gradients of FP32 segments; the FP64 form,
the spectra and the event positions are handed on in double precision.
"""
import math

import numpy as np
import torch

from paper_1204_5041_amd import autograd as AG
from paper_1204_5041_amd import binding as B

FLOP_PER_PAIR = 36          # Eq. (1)-(2) per (pixel, segment) pair
FLOP_PER_PAIR_BACK = 67     # its adjoint
FLOP_PER_PAIR_FLAT = 10     # the flat-sky form
EXACT_PAIRS = 3e10          # pairs above which the 64-bit sums take too long
EXACT_PAIRS_BACK = 1.2e10


def listed():
    return [
        # The plain map: Nside 64, one box of 2,000 FP64 segments around the
        # observer, a new box on every pass; the smallest call, whose cost is
        # latency, launches and planning.
        {"name": "render_fp64_nside64", "kind": "render", "form": "fp64", "nside": 64,
         "nseg": 2000, "seg64": True, "near": True},
        # The reference form at an ordinary size: one distant box a pass.
        {"name": "render_fp64_nside512", "kind": "render", "form": "fp64", "nside": 512,
         "nseg": 50000, "seg64": False, "near": False},
        # The headline map: Nside 2048, one box of FP32 segments per pass
        # (fewer than the benchmark's 400,000, the same rate per pair).
        {"name": "render_fp32c_nside2048", "kind": "render", "form": "fp32c", "nside": 2048,
         "nseg": 50000, "seg64": False, "near": False},
        # Boxes of very different sizes, each seen by its own cap of the sky,
        # in one launch; the sky keeps its boxes and is rendered again.
        {"name": "caps_nside1024", "kind": "caps", "nside": 1024, "nbox": 64, "median": 5000},
        # One step of fitting segments to a map: the differentiable map, a
        # quadratic loss and the gradients of every segment.
        {"name": "grad_nside256", "kind": "grad", "nside": 256, "nbox": 8, "nseg": 1500},
        # Eq. (1) at a catalogue of directions.
        {"name": "dirs_1003", "kind": "dirs", "form": "fp32c", "n": 1003, "nseg": 100000},
        # Stacked simulation boxes: 96 cones of the Nside 16 stacking grid,
        # looked at in a coarse map, where the light-cone stage counts.
        {"name": "stack_nside32", "kind": "stack", "nside": 32, "nside_c": 16, "cones": 96,
         "nseg": 20000, "snapshot": False},
        # The flat-sky patch of 7.2 degrees at 1024^2 pixels.
        {"name": "flat_1024", "kind": "flat", "nx": 1024, "ny": 1024, "nseg": 200000},
        # Power spectra: a small map, the benchmark's, and one of the
        # resolution of the full-sky string maps.
        {"name": "alm_nside128", "kind": "alm", "nside": 128, "lmax": 300},
        {"name": "alm_nside2048", "kind": "alm", "nside": 2048, "lmax": 4096},
        {"name": "alm_nside4096", "kind": "alm", "nside": 4096, "lmax": 6000},
        # Recording the light-cone events of one slab of a simulation.
        {"name": "events_25M", "kind": "events", "n": 25_600_000, "seg64": False},
    ]


def _log(rng, lo, hi):
    """A whole number spread evenly over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["render", "render", "shell", "caps", "grad", "dirs", "stack", "flat",
                       "alm", "alm", "events"])
    if kind == "render":
        form = rng.choice(["fp64", "fp32c"])
        nside = rng.choice([16, 32, 64, 128, 256, 512, 1024, 2048, _log(rng, 8, 1000)])
        top = (1.5e11 if form == "fp64" else 8e11) / (12 * nside * nside)
        nseg = _log(rng, 300, int(max(400, min(400_000, top))))
        return {"kind": kind, "form": form, "nside": nside, "nseg": nseg,
                "seg64": form == "fp64" and rng.random() < 0.5, "near": rng.random() < 0.3}
    if kind == "shell":
        nside = rng.choice([32, 64, 128, 256, 512])
        return {"kind": kind, "form": rng.choice(["fp64", "fp32c"]), "nside": nside,
                "nseg": _log(rng, 200, 20_000)}
    if kind == "caps":
        return {"kind": kind, "nside": rng.choice([64, 96, 256, 512, 1024, 2048]),
                "nbox": _log(rng, 8, 128), "median": _log(rng, 500, 5000)}
    if kind == "grad":
        nside = rng.choice([8, 16, 32, 64, 128, 256, 512])
        nbox = rng.randint(1, 8)
        top = 5e10 / (12 * nside * nside) / nbox
        return {"kind": kind, "nside": nside, "nbox": nbox,
                "nseg": _log(rng, 50, int(max(60, min(50_000, top))))}
    if kind == "dirs":
        n = _log(rng, 1, 1_000_000)
        return {"kind": kind, "form": rng.choice(["fp64", "fp32c"]), "n": n,
                "nseg": _log(rng, 1000, int(min(400_000, max(2000, 1e11 / n))))}
    if kind == "stack":
        nside_c = rng.choice([1, 16])
        return {"kind": kind, "nside": rng.choice([8, 16, 32, 64]), "nside_c": nside_c,
                "cones": 12 if nside_c == 1 else _log(rng, 12, 200),
                "nseg": _log(rng, 1000, 40_000), "snapshot": rng.random() < 0.3}
    if kind == "flat":
        nx = _log(rng, 32, 1500)
        ny = max(1, int(nx * rng.choice([1.0, 1.0, 0.5, 0.03])))
        return {"kind": kind, "nx": nx, "ny": ny, "nseg": _log(rng, 1000, 400_000)}
    if kind == "alm":
        nside = rng.choice([16, 32, 64, 128, 256, 512, 1024, 2048, 4096, _log(rng, 5, 400)])
        top = 1.45 if nside == 4096 else 3.0
        lmax = int(nside * rng.choice([1.0, top, rng.uniform(0.5, top), rng.uniform(0.5, top)]))
        return {"kind": kind, "nside": nside, "lmax": max(2, lmax - rng.choice([0, 1]))}
    return {"kind": kind, "n": _log(rng, 1000, 25_600_000), "seg64": rng.random() < 0.3}


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------
def _gen(seed, salt):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1_000_003 + salt) % (1 << 62))


def _unit(v):
    return v / v.norm(dim=1, keepdim=True)


def _u(g, n, lo=0.0, hi=1.0):
    return lo + (hi - lo) * torch.rand(n, dtype=torch.float64, device="cuda", generator=g)


def _segments(n, g, dtype, side=1.0, vmin=0.2, vmax=0.8):
    """x_rel, Xdot, X', dsigma: positions uniform in the box, Xdot.X' = 0 and
    Xdot^2 + X'^2 = 1."""
    n3 = dict(dtype=torch.float64, device="cuda", generator=g)
    x = torch.rand((n, 3), **n3) * side
    s = _unit(torch.randn((n, 3), **n3))
    h = torch.randn((n, 3), **n3)
    h = _unit(h - (h * s).sum(1, keepdim=True) * s)
    v = _u(g, n, vmin, vmax)
    ds = _u(g, n, 0.001, 0.01)
    out = (x, v[:, None] * h, (1.0 - v * v).sqrt()[:, None] * s, ds)
    return tuple(t.to(dtype).contiguous() for t in out)


def _directions(n, g):
    return _unit(torch.randn((n, 3), dtype=torch.float64, device="cuda", generator=g))


_KEYS = ("x_rel", "xdot", "xprime", "dsigma")


def _box(seg, **geom):
    return dict(zip(_KEYS, seg), **geom)


def _shell_centres():
    pts = set()
    for a in (1, -1):
        for b in (2, -2):
            for p in ((0, a, b), (0, b, a), (a, 0, b), (a, b, 0), (b, 0, a), (b, a, 0)):
                pts.add(p)
    return sorted(pts)


def _inputs(case, seed):
    """(eta0, boxes) of a case that sums over boxes."""
    kind = case["kind"]
    g = _gen(seed, 1)
    if kind in ("render", "dirs"):
        dtype = torch.float64 if case.get("seg64") else torch.float32
        if case.get("near"):   # a box around the observer
            return 1.0, [_box(_segments(case["nseg"], g, dtype), origin=(-0.5, -0.5, -0.5),
                              eta_lo=0.0, eta_hi=1.0)]
        d = _directions(1, g)[0].tolist()
        r = 0.1 * 140.0 ** float(_u(g, 1)) + math.sqrt(3.0) / 2.0
        return 16.0, [_box(_segments(case["nseg"], g, dtype),
                           origin=tuple(r * c - 0.5 for c in d), eta_lo=0.0, eta_hi=16.0)]
    if kind == "shell":
        # The 24 unit boxes of a shell, each a little off its place so that
        # no ray runs along an edge.
        return 3.0, [_box(_segments(case["nseg"], g, torch.float32),
                          origin=tuple(c - 0.5 + e for c, e in
                                       zip(p, _u(g, 3, -0.01, 0.01).tolist())),
                          eta_lo=0.4, eta_hi=1.1, vis=B.CSMAP_VIS_BOX, ext=(1.0, 1.0, 1.0))
                     for p in _shell_centres()]
    if kind == "caps":
        nbox = case["nbox"]
        spread = torch.randn(nbox, dtype=torch.float64, device="cuda", generator=g)
        count = (case["median"] * spread.exp()).round().clamp(100, 40 * case["median"]).tolist()
        r = (_u(g, nbox, math.log(0.1), math.log(14.0)).exp() + math.sqrt(3.0) / 2.0).tolist()
        frac = _u(g, nbox, math.log(0.001), math.log(0.05)).exp().tolist()
        dirs = _directions(nbox, g).tolist()
        boxes = []
        for b in range(nbox):
            boxes.append(_box(_segments(int(count[b]), g, torch.float32),
                              origin=tuple(r[b] * c - 0.5 for c in dirs[b]), eta_lo=0.0,
                              eta_hi=16.0, vis=B.CSMAP_VIS_CAP, cap_dir=tuple(dirs[b]),
                              cap_cos=1.0 - 2.0 * frac[b]))
        return 16.0, boxes
    if kind == "grad":
        dirs = _directions(case["nbox"], g).tolist()
        return 16.0, [_box(_segments(case["nseg"], g, torch.float32),
                           origin=tuple((b + 1 + math.sqrt(3.0) / 2.0) * c - 0.5
                                        for c in dirs[b]), eta_lo=0.0, eta_hi=16.0)
                      for b in range(case["nbox"])]
    if kind == "stack":
        high = case["nside_c"] == 16
        r_in, r_out, side = (13.4, 15.5, 2.4) if high else (1.4, 13.4, 16.0)
        pixels = torch.randperm(12 * case["nside_c"] ** 2, device="cuda",
                                generator=g)[:case["cones"]].tolist()
        # One run fills three cones, one per box axis; the speeds of
        # snapshot boxes reach the light cone at different times.
        runs = [_segments(case["nseg"], g, torch.float32, side)
                for _ in range((case["cones"] + 2) // 3)]
        boxes = []
        for k, pix in enumerate(pixels):
            cone, origin, _ = B.cone_place(case["nside_c"], pix, k % 3, r_in, r_out, side)
            boxes.append(_box(runs[k // 3], origin=tuple(float(v) for v in origin),
                              eta_lo=16.0 - r_out, eta_hi=16.0 - r_in,
                              snapshot=case["snapshot"], cone=cone))
        return 16.0, boxes
    if kind == "flat":
        n = case["nseg"]
        seg = _segments(n, g, torch.float64)
        cz = _u(g, n, math.cos(math.radians(6.0)), 1.0)
        ph = _u(g, n, 0.0, 2.0 * math.pi)
        r = _u(g, n, 1.4 ** 3, 15.5 ** 3).pow(1.0 / 3.0)
        st = (1.0 - cz * cz).sqrt()
        P = torch.stack([st * ph.cos(), st * ph.sin(), cz], 1) * r[:, None]
        seg = tuple(t.float().contiguous() for t in (P,) + seg[1:])
        return 16.0, [_box(seg, origin=(0.0, 0.0, 0.0), eta_lo=0.5, eta_hi=14.6)]
    raise ValueError(kind)


def _patch(case):
    return dict(center=(0.0, 0.0, 1.0), e1=(1.0, 0.0, 0.0), e2=(0.0, 1.0, 0.0), nx=case["nx"],
                ny=case["ny"], pix=math.radians(7.2) / max(case["nx"], case["ny"]),
                accept_cos=math.cos(math.radians(6.0)))


def _map_input(case, seed):
    """A sky map with power on every scale: pixel noise over a smooth part."""
    g = _gen(seed, 2)
    npix = 12 * case["nside"] ** 2
    ramp = torch.linspace(-1.0, 1.0, npix, dtype=torch.float64, device="cuda")
    return torch.randn(npix, dtype=torch.float64, device="cuda", generator=g) + 3.0 * ramp * ramp


def _event_input(case, seed):
    g = _gen(seed, 3)
    seg = _segments(case["n"], g, torch.float64 if case["seg64"] else torch.float32, 1.0, 0.0,
                    0.95)
    return dict(x_rel=seg[0], xdot=seg[1], origin=(3.7, -2.1, 1.4), eta0=16.0, eta_lo=11.0,
                eta_hi=11.6)


_FORMS = {"fp64": B.CSMAP_FORM_FP64, "fp32c": B.CSMAP_FORM_FP32C}


def _add(sky, boxes):
    for bx in boxes:
        sky.add_box(**bx)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "alm":
        return {"case": case, "map": _map_input(case, seed)}
    if kind == "events":
        return {"case": case, "in": _event_input(case, seed)}
    eta0, boxes = _inputs(case, seed)
    nside = case.get("nside", 64)
    st = {"case": case, "boxes": boxes,
          "sky": B.Sky(nside, eta0, _FORMS[case.get("form", "fp32c")])}
    if kind in ("caps", "dirs", "stack", "flat"):   # the sky keeps these boxes
        _add(st["sky"], boxes)
    if kind == "dirs":
        st["xyz"] = 3.0 * _directions(case["n"], _gen(seed, 4))
    if kind == "grad":
        g = _gen(seed, 5)
        st["w"] = torch.randn(12 * nside * nside, dtype=torch.float64, device="cuda", generator=g)
        for bx in boxes:
            for k in _KEYS:
                bx[k].requires_grad_(True)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "alm":
        alm = B.map2alm(st["map"], case["lmax"])
        return {"alm": alm, "cl": B.alm2cl(alm, case["lmax"])}
    if kind == "events":
        pos, delta, keep = B.cone_events(**st["in"])
        return {"pos": pos, "delta": delta, "keep": keep}
    sky = st["sky"]
    if kind in ("render", "shell"):
        # The next box or batch of boxes: drop the last one, add, render.
        sky.reset()
        _add(sky, st["boxes"])
        m = sky.render()
        return m if case["form"] == "fp64" else m.float()
    if kind in ("caps", "stack"):
        return sky.render().float()
    if kind == "dirs":
        v = sky.render_dirs(st["xyz"])
        return v if case["form"] == "fp64" else v.float()
    if kind == "flat":
        return sky.render_flat(**_patch(case)).float()
    m = AG.render(sky, st["boxes"])
    loss = (st["w"] * m * m).sum()
    leaves = [bx[k] for bx in st["boxes"] for k in _KEYS]
    grads = torch.autograd.grad(loss, leaves)
    return {"map": m.detach().float(), "grads": list(grads)}


# ---------------------------------------------------------------------------
# What a pass cannot do without.
# ---------------------------------------------------------------------------
def _pairs(case):
    """(segments read, pixels written, pairs); averages for drawn boxes."""
    kind = case["kind"]
    npix = 12 * case.get("nside", 64) ** 2
    if kind == "render":
        return case["nseg"], npix, npix * case["nseg"]
    if kind == "dirs":
        return case["nseg"], case["n"], case["n"] * case["nseg"]
    if kind == "shell":   # a box is seen by about 1/14 of the sky, 83% of its segments kept
        return 24 * case["nseg"], npix, 24 * 0.83 * case["nseg"] * npix / 14
    if kind == "caps":    # mean of the counts and of the sky fractions
        n = case["nbox"] * case["median"] * math.exp(0.5)
        return n, npix, n * npix * 0.0125
    if kind == "grad":
        n = case["nbox"] * case["nseg"]
        return n, npix, n * npix
    if kind == "stack":   # the share of a box inside its cone and slab
        n = case["cones"] * case["nseg"]
        return n, npix, 0.13 * n * npix
    return case["nseg"], case["nx"] * case["ny"], case["nseg"] * 0.75 * case["nx"] * case["ny"]


def work(case):
    kind = case["kind"]
    if kind == "events":
        e = 8 if case["seg64"] else 4
        return {"bytes": case["n"] * (6 * e + 33), "flops": 60 * case["n"]}
    if kind == "alm":
        nside, lmax = case["nside"], case["lmax"]
        size = (lmax + 1) * (lmax + 2) // 2
        # Ring transforms (5 n log2 n for each ring's real samples, half of a
        # complex transform) and 8 per (l, m, ring pair).
        fft = 12 * nside * nside * 2.5 * math.log2(4 * nside)
        return {"bytes": 8 * 12 * nside * nside + 16 * size, "flops": fft + 8.0 * size * 2 * nside}
    nseg, npix, pairs = _pairs(case)
    e = 8 if case.get("seg64") else 4
    bytes_ = 10 * e * nseg + 8 * npix
    if kind == "flat":
        return {"bytes": bytes_, "flops": FLOP_PER_PAIR_FLAT * pairs}
    if kind == "grad":
        return {"bytes": bytes_ + 8 * npix + 10 * e * nseg,
                "flops": (FLOP_PER_PAIR + FLOP_PER_PAIR_BACK) * pairs}
    if kind == "dirs":
        bytes_ += 24 * npix
    return {"bytes": bytes_, "flops": FLOP_PER_PAIR * pairs}


# ---------------------------------------------------------------------------
# The outputs in 64 bits.
# ---------------------------------------------------------------------------
def _pix2vec(nside):
    """Pixel centres of a RING map (Gorski et al. 2005), (npix, 3)."""
    N = nside
    p = torch.arange(12 * N * N, device="cuda", dtype=torch.int64)
    ncap = 2 * N * (N - 1)

    def cap(q):   # ring and position of index q counted from a pole
        i = ((1.0 + (1.0 + 2.0 * q.double()).sqrt()) / 2.0).floor().long()
        i = torch.where(2 * i * (i - 1) > q, i - 1, i)
        i = torch.where(2 * i * (i + 1) <= q, i + 1, i)
        return i, q - 2 * i * (i - 1)

    north, south = p < ncap, p >= 12 * N * N - ncap
    qs = 12 * N * N - 1 - p
    ic, jc = cap(torch.where(south, qs, torch.where(north, p, torch.zeros_like(p))))
    jc = torch.where(south, 4 * ic - 1 - jc, jc)
    b = (p - ncap).clamp(0, max(0, 12 * N * N - 2 * ncap - 1))
    ib, jb = b // (4 * N) + N, b % (4 * N)
    incap = north | south
    fr = (ic.double() / N) ** 2 / 3.0
    zc = torch.where(south, fr - 1.0, 1.0 - fr)
    sc = (fr * (2.0 - fr)).sqrt()
    zb = (4 * N - 2 * ib).double() / (3.0 * N)
    z = torch.where(incap, zc, zb)
    s = torch.where(incap, sc, ((1.0 - zb) * (1.0 + zb)).sqrt())
    phi = torch.where(incap, (jc.double() + 0.5) * (math.pi / 2) / ic.clamp(min=1).double(),
                      (jb.double() + 0.5 * ((ib - N) % 2 == 0).double()) * (math.pi / 2) / N)
    return torch.stack([s * phi.cos(), s * phi.sin(), z], 1)


def _ang2pix(nside, v):
    n = v / v.norm(dim=1, keepdim=True)
    z, za = n[:, 2], n[:, 2].abs()
    tt = torch.remainder(torch.atan2(n[:, 1], n[:, 0]) / (math.pi / 2), 4.0)
    N = nside
    a, c = N * (0.5 + tt), N * z * 0.75
    jp, jm = (a - c).floor().long(), (a + c).floor().long()
    ir = N + 1 + jp - jm
    ip = torch.remainder((jp + jm - N + (1 - (ir & 1)) + 1) // 2, 4 * N)
    belt = 2 * N * (N - 1) + (ir - 1) * 4 * N + ip
    tp = tt - tt.floor()
    w = N * (3.0 * (1.0 - za)).sqrt()
    kp, km = (tp * w).floor().long(), ((1.0 - tp) * w).floor().long()
    ir = kp + km + 1
    ip = torch.remainder((tt * ir.double()).floor().long(), 4 * ir)
    cap = torch.where(z > 0, 2 * ir * (ir - 1) + ip, 12 * N * N - 2 * ir * (ir + 1) + ip)
    return torch.where(za <= 2.0 / 3.0, belt, cap)


def _crossing(P0, V, R0):
    vv = (V * V).sum(1)
    b = (P0 * V).sum(1) + R0
    r = P0.norm(dim=1)
    c = (r - R0) * (r + R0)
    q = -(b + torch.copysign((b * b - (vv - 1.0) * c).clamp(min=0.0).sqrt(), b))
    return torch.minimum(q / (vv - 1.0), c / q)


def _events_of(bx, eta0):
    """P, Xdot, X', dsigma of a box's events inside its slab (and cone)."""
    x, V, T, ds = (bx[k].double() for k in _KEYS)
    o = torch.tensor(bx["origin"], dtype=torch.float64, device="cuda")
    cone = bx.get("cone")
    if cone is not None:
        rot = torch.from_numpy(np.array(cone.rot[:]).reshape(3, 3)).cuda()
        x, V, T = (torch.stack([(t * rot[k]).sum(1) for k in range(3)], 1) for t in (x, V, T))
    P = o + x
    if bx.get("snapshot"):
        D = _crossing(P, V, eta0 - bx["eta_lo"])
        keep = (D >= 0) & (D < bx["eta_hi"] - bx["eta_lo"])
        P = P + V * D[:, None]
    else:
        eta = eta0 - P.norm(dim=1)
        keep = (eta >= bx["eta_lo"]) & (eta < bx["eta_hi"])
    if cone is not None and cone.nside > 0:
        keep = keep & (_ang2pix(cone.nside, P) == cone.pix)
    return (t[keep] for t in (P, V, T, ds))


def _sees(bx, n, eta0):
    vis = bx.get("vis", B.CSMAP_VIS_ALL)
    if vis == B.CSMAP_VIS_CAP:
        c = bx["cap_dir"]
        return (n[:, 0] * c[0] + n[:, 1] * c[1]) + n[:, 2] * c[2] >= bx["cap_cos"]
    if vis == B.CSMAP_VIS_BOX:
        o = torch.tensor(bx["origin"], dtype=torch.float64, device="cuda")
        ta, tb = o / n, (o + torch.tensor(bx["ext"], dtype=torch.float64, device="cuda")) / n
        t_in = torch.minimum(ta, tb).max(1).values.clamp(min=0.0)
        t_out = torch.maximum(ta, tb).min(1).values
        return (t_in <= t_out) & (t_out > eta0 - bx["eta_hi"]) & (t_in <= eta0 - bx["eta_lo"])
    return None


def _theta(n, P, V, T, ds):
    """Sum over segments of Eq. (1) at the directions n."""
    R = P.norm(dim=1)
    H = P / R[:, None]
    eps = ((T * T).sum(1) / (1.0 - (V * V).sum(1))).sqrt()
    d = [n[:, k, None] - H[None, :, k] for k in range(3)]
    a = n[:, 0, None] * T[:, 0] + n[:, 1, None] * T[:, 1] + n[:, 2, None] * T[:, 2]
    b = 1.0 + n[:, 0, None] * V[:, 0] + n[:, 1, None] * V[:, 1] + n[:, 2, None] * V[:, 2]
    q = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
    vd = V[:, 0] * d[0] + V[:, 1] * d[1] + V[:, 2] * d[2]
    td = T[:, 0] * d[0] + T[:, 1] * d[1] + T[:, 2] * d[2]
    return ((vd - a * td / b) / q) @ (-4.0 * eps * ds / R)


def _exact_map(n, eta0, boxes):
    out = torch.zeros(n.shape[0], dtype=torch.float64, device="cuda")
    for bx in boxes:
        P, V, T, ds = _events_of(bx, eta0)
        see = _sees(bx, n, eta0)
        at = torch.arange(n.shape[0], device="cuda") if see is None else see.nonzero()[:, 0]
        cs = max(1, min(len(ds), 4096))
        cp = max(1, (1 << 24) // cs)
        for p in range(0, len(at), cp):
            i = at[p:p + cp]
            for s in range(0, len(ds), cs):
                out[i] += _theta(n[i], P[s:s + cs], V[s:s + cs], T[s:s + cs], ds[s:s + cs])
    return out


def _exact_grads(n, eta0, boxes, cot):
    grads = []
    for bx in boxes:
        leaf = [bx[k].detach().double().requires_grad_(True) for k in _KEYS]
        o = torch.tensor(bx["origin"], dtype=torch.float64, device="cuda")
        total = [torch.zeros_like(t) for t in leaf]
        cp = max(1, (1 << 24) // max(1, len(leaf[3])))
        for p in range(0, n.shape[0], cp):
            t = (_theta(n[p:p + cp], o + leaf[0], *leaf[1:]) * cot[p:p + cp]).sum()
            for k, gk in enumerate(torch.autograd.grad(t, leaf)):
                total[k] += gk
        grads += total
    return grads


def _exact_alm(case, seed):
    N, lmax = case["nside"], case["lmax"]
    hmap = _map_input(case, seed)
    nring = 4 * N - 1
    m = torch.arange(lmax + 1, device="cuda")
    F = torch.zeros((nring, lmax + 1), dtype=torch.complex128, device="cuda")
    z = torch.zeros(nring, dtype=torch.float64, device="cuda")
    first = 0
    for i in range(1, nring + 1):
        length = 4 * min(i, N, 4 * N - i)
        x = torch.fft.fft(hmap[first:first + length])[m % length]
        k = min(i, 4 * N - i)
        half = 0.5 if k < N or (i - N) % 2 == 0 else 0.0
        zi = 1.0 - k * k / (3.0 * N * N) if k < N else (4 * N - 2 * i) / (3.0 * N)
        z[i - 1] = -zi if k < N and i > 2 * N else zi
        turn = torch.remainder(m.double() * half, float(length)) * (-2.0 * math.pi / length)
        F[i - 1] = x * torch.polar(torch.ones_like(turn), turn)
        first += length
    md = m.double()
    # lambda_mm through its logarithm; l runs over all m at once.
    lg = torch.cat([torch.zeros(1, dtype=torch.float64, device="cuda"),
                    (0.5 * torch.log((2 * md[1:] + 1) / (2 * md[1:]))).cumsum(0)])
    # (1 - z)(1 + z) from the ring numbers, exact near the poles.
    ring = torch.arange(1, nring + 1, device="cuda", dtype=torch.float64)
    k = torch.minimum(ring, 4.0 * N - ring)
    fr = (k / N) ** 2 / 3.0
    s2 = torch.where(k < N, fr * (2.0 - fr), (1.0 - z) * (1.0 + z))
    sign = 1.0 - 2.0 * (m % 2).double()
    mm = sign * torch.exp(lg + 0.5 * torch.log(s2)[:, None] * md) / math.sqrt(4.0 * math.pi)
    cur, prev = torch.zeros_like(mm), torch.zeros_like(mm)
    w = 4.0 * math.pi / (12 * N * N)
    out = torch.zeros((lmax + 1) * (lmax + 2) // 2, dtype=torch.complex128, device="cuda")
    for l in range(lmax + 1):
        a = torch.sqrt((4.0 * l * l - 1.0) / (l * l - md[:l] * md[:l]))
        b = torch.sqrt(((l - 1.0) ** 2 - md[:l] * md[:l]).clamp(min=0.0) /
                       (4.0 * (l - 1.0) ** 2 - 1.0))
        new = a * (z[:, None] * cur[:, :l] - b * prev[:, :l])
        prev[:, :l] = cur[:, :l]
        cur[:, :l] = new
        cur[:, l] = mm[:, l]
        c = cur[:, :l + 1]
        s = torch.complex((c * F.real[:, :l + 1]).sum(0), (c * F.imag[:, :l + 1]).sum(0))
        out[m[:l + 1] * (2 * lmax + 1 - m[:l + 1]) // 2 + l] = w * s
    cl = torch.zeros(lmax + 1, dtype=torch.float64, device="cuda")
    for l in range(lmax + 1):
        p = out[m[:l + 1] * (2 * lmax + 1 - m[:l + 1]) // 2 + l].abs() ** 2
        cl[l] = (2.0 * p.sum() - p[0]) / (2 * l + 1)
    return {"alm": out, "cl": cl}


def exact(case, seed):
    kind = case["kind"]
    if kind == "alm":
        if case["nside"] > 512 or case["lmax"] > 1100:
            return None
        return _exact_alm(case, seed)
    if kind == "events":
        e = _event_input(case, seed)
        P0 = torch.tensor(e["origin"], dtype=torch.float64, device="cuda") + e["x_rel"].double()
        V = e["xdot"].double()
        D = _crossing(P0, V, e["eta0"] - e["eta_lo"])
        keep = (D >= 0) & (D < e["eta_hi"] - e["eta_lo"])
        nan = torch.full_like(D, float("nan"))
        return {"pos": torch.where(keep[:, None], P0 + V * D[:, None], nan[:, None]),
                "delta": torch.where(keep, D, nan), "keep": None}
    pairs = _pairs(case)[2]
    if pairs > (EXACT_PAIRS_BACK if kind == "grad" else EXACT_PAIRS):
        return None
    eta0, boxes = _inputs(case, seed)
    if kind == "flat":
        return _exact_flat(case, eta0, boxes[0])
    if kind == "dirs":
        n = _unit(3.0 * _directions(case["n"], _gen(seed, 4)))
        return _exact_map(n, eta0, boxes)
    n = _pix2vec(case["nside"])
    theta = _exact_map(n, eta0, boxes)
    if kind != "grad":
        return theta
    w = torch.randn(n.shape[0], dtype=torch.float64, device="cuda", generator=_gen(seed, 5))
    return {"map": theta, "grads": _exact_grads(n, eta0, boxes, 2.0 * w * theta)}


def _exact_flat(case, eta0, bx):
    p = _patch(case)
    P, V, T, ds = _events_of(bx, eta0)
    D = P[:, 2]
    ok = (D > 0) & (D > p["accept_cos"] * P.norm(dim=1))
    P, V, T, ds, D = P[ok], V[ok], T[ok], ds[ok], D[ok]
    eps = ((T * T).sum(1) / (1.0 - (V * V).sum(1))).sqrt()
    u = V - (T[:, 2] / (1.0 + V[:, 2]))[:, None] * T
    k = -4.0 * eps * ds / D / p["pix"]
    s = P[:, :2] / D[:, None] / p["pix"]
    x = torch.arange(p["nx"], dtype=torch.float64, device="cuda") + 0.5 - 0.5 * p["nx"]
    y = torch.arange(p["ny"], dtype=torch.float64, device="cuda") + 0.5 - 0.5 * p["ny"]
    out = torch.zeros((p["ny"], p["nx"]), dtype=torch.float64, device="cuda")
    cs = 2048
    cy = max(1, (1 << 24) // (cs * p["nx"]))
    for c in range(0, len(ds), cs):
        e = slice(c, c + cs)
        dx = x[None, :, None] - s[None, None, e, 0]
        for r in range(0, p["ny"], cy):
            dy = y[r:r + cy, None, None] - s[None, None, e, 1]
            q = dx * dx + dy * dy
            out[r:r + cy] += (((k * u[:, 0])[e] * dx + (k * u[:, 1])[e] * dy) / q).sum(-1)
    return out
