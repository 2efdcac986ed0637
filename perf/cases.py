"""Workloads of the library's public entry points, for timing them.

A case is a dict of plain values.  ``prepare`` makes what a program has in
hand before the call (a stack, offsets, output buffers it keeps), ``run`` is
one pass through the entry point, ``work`` the bytes and operations the pass
cannot do without, and ``exact`` the same outputs in 64 bits, written from
the definitions with torch alone.

Kinds of case:
  forward   deskew(): volume and projections, or the projections alone, from a
            uniform scan or from measured offsets per image
  view      view(): the rotated projections
  rolling   RollingView.update(): one call per camera image
  autograd  deskew_volume() and its backward, one calibration step
  affine    affine(): the real-space grid
  jobs      JobLauncher.launch(): many stacks of different sizes in one call
"""
import math

import numpy as np
import torch

import paper_2211_00645_amd as dsk
from paper_2211_00645_amd import autograd, synth
from paper_2211_00645_amd.batch import JobLauncher, plan_job
from paper_2211_00645_amd.rolling import RollingView

PIXEL = 0.115          # sample-space pixel, um
DEV = "cuda"


def listed():
    return [
        # the whole stack of a live acquisition: volume and both projections
        # into buffers the program keeps
        dict(name="live_stack", kind="forward", planes=512, rows=512, cols=2048, angle=35.0,
             step=0.4, vol=True, jitter=0.0, f32=False, keep=True, jobs=0, scale=0.0),
        # the smallest stack that is deskewed as such: latency and launches
        dict(name="small_stack", kind="forward", planes=64, rows=128, cols=256, angle=30.0,
             step=0.4, vol=True, jitter=0.0, f32=False, keep=False, jobs=0, scale=0.0),
        # a region of interest cut to the sample, no side a round number, at
        # the stage's measured positions
        dict(name="odd_region", kind="forward", planes=201, rows=487, cols=1531, angle=45.0,
             step=0.31, vol=True, jitter=0.3, f32=False, keep=True, jobs=0, scale=0.0),
        # the live widefield-like view: projections only, the volume not kept
        dict(name="live_view", kind="forward", planes=512, rows=512, cols=2048, angle=35.0,
             step=0.4, vol=False, jitter=0.0, f32=False, keep=True, jobs=0, scale=0.0),
        # the display of the narrow live region: 50 images of 1304 x 87 pixels
        # spread over 3652
        dict(name="live_region", kind="forward", planes=50, rows=1304, cols=87, angle=35.0,
             step=10.2143, vol=False, jitter=0.0, f32=False, keep=False, jobs=0, scale=0.0),
        # the live view turned to look down the optical axis
        dict(name="top_view", kind="view", planes=512, rows=512, cols=2048, angle=35.0, step=0.4,
             vol=False, jitter=0.0, f32=False, keep=True, jobs=0, scale=0.0),
        # dim samples: the view refreshed after every image, here 8 images of
        # one scan and the same 8 of the next
        dict(name="rolling_view", kind="rolling", planes=512, rows=512, cols=2048, angle=35.0,
             step=0.4, vol=True, jitter=0.0, f32=False, keep=True, jobs=8, scale=0.0),
        # one step of the sheet-angle calibration at its full size
        dict(name="calibration", kind="autograd", planes=256, rows=512, cols=1024, angle=30.0,
             step=0.4, vol=True, jitter=0.0, f32=True, keep=False, jobs=0, scale=0.0),
        # the same on the first images of a small crop
        dict(name="calibration_crop", kind="autograd", planes=37, rows=131, cols=517, angle=30.0,
             step=0.4, vol=True, jitter=0.0, f32=True, keep=False, jobs=0, scale=0.0),
        # the real-space grid of a whole stack, for analysis
        dict(name="affine_stack", kind="affine", planes=512, rows=512, cols=2048, angle=35.0,
             step=0.4, vol=True, jitter=0.0, f32=False, keep=True, jobs=0, scale=0.0),
        # the same of an odd crop scanned finely
        dict(name="affine_fine", kind="affine", planes=150, rows=203, cols=1001, angle=45.0,
             step=0.2, vol=True, jitter=0.0, f32=False, keep=False, jobs=0, scale=0.0),
        # what the serving loop sends out together: stacks of many sizes
        dict(name="many_stacks", kind="jobs", planes=0, rows=0, cols=0, angle=0.0, step=0.0,
             vol=True, jitter=0.0, f32=False, keep=True, jobs=20, scale=0.25),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["forward", "forward", "forward", "view", "rolling", "autograd",
                           "affine", "jobs"])
        c = dict(kind=kind, planes=log(16, 512), rows=log(48, 1304), cols=log(87, 2048),
                 angle=rng.choice([30.0, 35.0, 45.0]), step=round(rng.uniform(0.2, 0.8), 4),
                 vol=True, jitter=0.0, f32=False, keep=rng.random() < 0.5, jobs=0, scale=0.0)
        if rng.random() < 0.5:          # a camera's round region
            c["rows"] = max(64, c["rows"] // 64 * 64)
            c["cols"] = max(64, c["cols"] // 64 * 64)
        if kind == "forward":
            c["vol"] = rng.random() < 0.6
            c["jitter"] = rng.choice([0.0, 0.3])
            c["f32"] = rng.random() < 0.25
        elif kind == "view":
            c["vol"] = False
        elif kind == "rolling":
            c["planes"], c["jobs"] = max(32, c["planes"]), rng.choice([4, 8, 16])
        elif kind == "autograd":
            c["f32"] = True
        elif kind == "jobs":
            c.update(planes=0, rows=0, cols=0, angle=0.0, step=0.0,
                     jobs=log(4, 21), scale=round(rng.uniform(0.12, 0.3), 3))
        if 1e6 < work(c)["bytes"] < 5e9:
            return c


# ---------------------------------------------------------------- geometry

def _shift(c):
    return (c["step"] * math.cos(c["angle"] * math.pi / 180.0)) / PIXEL


def _offsets(c, seed):
    n = np.arange(c["planes"], dtype=np.float64)
    o = n * _shift(c)
    if c["jitter"]:
        o = o + np.random.default_rng(seed).normal(0.0, c["jitter"], c["planes"])
    return o


def _frame(o, cols):
    b = math.floor(o.min())
    return b, cols + math.ceil(o.max()) - b


def _fixed_frame(c):
    """The frame a program keeps while the offsets jitter: two columns more
    than the nominal scan's at each end."""
    b, w = _frame(_offsets(dict(c, jitter=0.0), 0), c["cols"])
    return (b - 2, w + 4) if c["jitter"] else (b, w)


def _view_geometry(c, theta=0.0):
    t, a = math.radians(theta), math.radians(c["angle"])
    k = math.cos(t - a)
    s = c["step"] * math.cos(t) / (PIXEL * k)
    o = np.arange(c["planes"], dtype=np.float64) * s
    b, w = _frame(o, c["cols"])
    return o, b, w, k, math.floor((w - 1) * k) + 1


def _affine_grid(c):
    pc = PIXEL * math.cos(c["angle"] * math.pi / 180.0)
    hi = (c["planes"] - 1) * c["step"] + (c["cols"] - 1) * pc
    return pc, math.floor(hi / PIXEL) + 1


def _job_shapes(c):
    return synth.ragged_jobs(c["jobs"], seed=c["jobs"], scale=c["scale"])


def work(c):
    n, r, k = c["planes"], c["rows"], c["cols"]
    if c["kind"] == "jobs":
        by = fl = 0
        for j in _job_shapes(c):
            w = work(dict(c, kind="forward", planes=j["planes"], rows=j["rows"], cols=j["cols"],
                          angle=j["angle_deg"], step=j["step_um"]))
            by, fl = by + w["bytes"], fl + w["flops"]
        return {"bytes": by, "flops": fl}
    if c["kind"] == "view":
        return {"bytes": 2 * n * r * k + 8 * r * _view_geometry(c)[4], "flops": 5 * n * r * k}
    if c["kind"] == "affine":
        ny = _affine_grid(c)[1]
        return {"bytes": 2 * n * r * k + 4 * ny * r * k, "flops": 3 * ny * r * k}
    if c["kind"] == "rolling":
        # per image: the image, and over the columns it reaches the old and
        # new deskewed image, the running sum and both projections
        band = 2 * r * k + (8 + 16 + 8) * r * (k + 1)
        return {"bytes": 2 * c["jobs"] * band, "flops": 2 * c["jobs"] * 6 * r * k}
    w = _fixed_frame(c)[1]
    if c["kind"] == "autograd":
        return {"bytes": 4 * n * r * k + 4 * n * r * w + 12 * n * r * k,
                "flops": 3 * n * r * w + 6 * n * r * k}
    by = (4 if c["f32"] else 2) * n * r * k + 8 * r * w + (4 * n * r * w if c["vol"] else 0)
    return {"bytes": by, "flops": 5 * n * r * k}


# ---------------------------------------------------------------- inputs

def _stack(shape, seed, f32=False):
    """A fluorescence stack: Poisson counts over a dim background with bright
    structure along all three axes."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    a, b, c = (torch.rand(s, generator=g, device=DEV).pow_(4) for s in shape)
    out = torch.empty(shape, dtype=torch.float32 if f32 else torch.uint16, device=DEV)
    step = max(1, (1 << 27) // (shape[1] * shape[2]))
    for p in range(0, shape[0], step):
        rate = 100.0 + 3000.0 * a[p:p + step, None, None] * b[None, :, None] * c[None, None, :]
        v = torch.poisson(rate, generator=g).clamp_(max=65535.0)
        out[p:p + step] = v if f32 else v.to(torch.int32).to(torch.uint16)
    return out


def _grad_volume(shape, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) + 77)
    return torch.randn(shape, generator=g, device=DEV)


def _rolling_images(c, seed):
    """The filled stack, the first image replaced, and the images of the two
    scans that come in."""
    n, r, k = c["planes"], c["rows"], c["cols"]
    return (_stack((n, r, k), seed), n // 3, _stack((c["jobs"], r, k), seed + 1000),
            _stack((c["jobs"], r, k), seed + 2000))


def prepare(c, seed):
    n, r, k = c["planes"], c["rows"], c["cols"]
    s = {"case": c}
    if c["kind"] == "jobs":
        s["stacks"], s["jobs"], s["out"] = [], [], []
        for i, j in enumerate(_job_shapes(c)):
            st = _stack((j["planes"], j["rows"], j["cols"]), seed + 101 * i)
            job, res = plan_job(st, j["angle_deg"], j["step_um"], j["pixel_um"])
            s["stacks"].append(st)
            s["jobs"].append(job)
            s["out"].append({x: res[x] for x in ("vol", "psum", "pmax")})
        s["launcher"] = JobLauncher(max_jobs=64)
        return s
    if c["kind"] == "rolling":
        st, first, one, two = _rolling_images(c, seed)
        s["view"] = RollingView(n, r, k, c["angle"], c["step"], PIXEL)
        for i in range(n):
            s["view"].update(i, st[i])
        s["first"] = first
        s["scans"] = [[x[i] for i in range(c["jobs"])] for x in (one, two)]
        return s
    s["stack"] = _stack((n, r, k), seed, c["f32"])
    if c["kind"] == "forward":
        o = _offsets(c, seed)
        s["origin"], s["width"] = _fixed_frame(c)
        s["offsets"] = torch.from_numpy(o).to(DEV) if c["jitter"] else None
        w = s["width"]
        if c["keep"]:
            s["out"] = {"psum": torch.empty((r, w), device=DEV), "pmax": torch.empty((r, w), device=DEV)}
            if c["vol"]:
                s["out"]["vol"] = torch.empty((n, r, w), device=DEV)
    elif c["kind"] == "view":
        s["workspace"] = torch.empty((2 * r * _view_geometry(c)[2],), device=DEV) if c["keep"] else None
    elif c["kind"] == "autograd":
        o = _offsets(c, seed)
        s["origin"], s["width"] = _frame(o, k)
        s["stack"].requires_grad_(True)
        s["offsets"] = torch.from_numpy(o).to(DEV).requires_grad_(True)
        s["grad"] = _grad_volume((n, r, s["width"]), seed)
    elif c["kind"] == "affine" and c["keep"]:
        s["out"] = torch.empty((_affine_grid(c)[1], r, k), device=DEV)
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    c = s["case"]
    if c["kind"] == "forward":
        if s["offsets"] is None:
            res = dsk.deskew(s["stack"], c["angle"], c["step"], PIXEL, vol=c["vol"],
                             out=s.get("out"))
        else:
            res = dsk.deskew(s["stack"], offsets=s["offsets"], origin=s["origin"],
                             width=s["width"], vol=c["vol"], out=s.get("out"))
        return {x: res[x] for x in ("vol", "psum", "pmax") if x in res}
    if c["kind"] == "view":
        res = dsk.view(s["stack"], 0.0, c["angle"], c["step"], PIXEL, workspace=s["workspace"])
        return {"vsum": res["vsum"], "vmax": res["vmax"]}
    if c["kind"] == "rolling":
        v = s["view"]
        for scan in s["scans"]:
            for i, image in enumerate(scan):
                v.update(s["first"] + i, image)
        return {"vol": v.vol, "sum64": v.sum64, "psum": v.psum, "pmax": v.pmax}
    if c["kind"] == "autograd":
        vol = autograd.deskew_volume(s["stack"], s["offsets"], s["origin"], s["width"])
        gs, go = torch.autograd.grad(vol, (s["stack"], s["offsets"]), s["grad"])
        return {"vol": vol, "grad_stack": gs, "grad_offsets": go}
    if c["kind"] == "affine":
        return dsk.affine(s["stack"], c["angle"], c["step"], PIXEL, out=s.get("out"))[0]
    s["launcher"].launch(s["jobs"])
    return s["out"]


# ---------------------------------------------------------------- in 64 bits

def _remap64(stack, o, b, w):
    n, r, k = stack.shape
    vol = torch.zeros((n, r, w), dtype=torch.float64, device=DEV)
    for i in range(n):
        t = float(o[i]) - b
        q = math.floor(t)
        f = t - q
        row = stack[i].double() if stack.dtype == torch.float32 else stack[i].to(torch.int32).double()
        for at, weight in ((q, 1.0 - f), (q + 1, f)):
            lo, hi = max(0, at), min(w, at + k)
            if lo < hi:
                vol[i, :, lo:hi] += weight * row[:, lo - at:hi - at]
    return vol


def _projections64(stack, o, b, w):
    v = _remap64(stack, o, b, w)
    return v, v.sum(0), v.amax(0)


def _stretch64(p, factor, width):
    u = torch.arange(width, dtype=torch.float64, device=DEV) / factor
    i = torch.floor(u)
    f, i = u - i, i.long()
    pad = torch.cat([p, torch.zeros((p.shape[0], 2), dtype=p.dtype, device=DEV)], 1)
    i = i.clamp(max=p.shape[1])
    return (1.0 - f) * pad[:, i] + f * pad[:, i + 1]


def exact(c, seed):
    n, r, k = c["planes"], c["rows"], c["cols"]
    if c["kind"] == "jobs":
        res = []
        for i, j in enumerate(_job_shapes(c)):
            d = dict(c, planes=j["planes"], cols=j["cols"], angle=j["angle_deg"], step=j["step_um"])
            o = _offsets(d, seed)
            v, ps, pm = _projections64(_stack((j["planes"], j["rows"], j["cols"]), seed + 101 * i),
                                       o, *_frame(o, j["cols"]))
            res.append({"vol": v, "psum": ps, "pmax": pm})
        return res
    if c["kind"] == "rolling":
        st, first, _, two = _rolling_images(c, seed)
        st[first:first + c["jobs"]] = two
        o = _offsets(c, seed)
        v, ps, pm = _projections64(st, o, *_frame(o, k))
        return {"vol": v, "sum64": ps, "psum": ps, "pmax": pm}
    st = _stack((n, r, k), seed, c["f32"])
    if c["kind"] == "forward":
        o = _offsets(c, seed)
        v, ps, pm = _projections64(st, o, *_fixed_frame(c))
        return {"vol": v, "psum": ps, "pmax": pm} if c["vol"] else {"psum": ps, "pmax": pm}
    if c["kind"] == "view":
        o, b, w, factor, width = _view_geometry(c)
        _, ps, pm = _projections64(st, o, b, w)
        return {"vsum": _stretch64(ps, factor, width), "vmax": _stretch64(pm, factor, width)}
    if c["kind"] == "autograd":
        o = _offsets(c, seed)
        b, w = _frame(o, k)
        grad = _grad_volume((n, r, w), seed)
        gs = torch.zeros((n, r, k), dtype=torch.float64, device=DEV)
        go = torch.zeros((n,), dtype=torch.float64, device=DEV)
        for i in range(n):
            q = math.floor(float(o[i]) - b)
            f = float(o[i]) - b - q
            g = torch.cat([grad[i].double(), torch.zeros((r, 2), dtype=torch.float64, device=DEV)], 1)
            g0, g1 = g[:, q:q + k], g[:, q + 1:q + 1 + k]
            gs[i] = (1.0 - f) * g0 + f * g1
            go[i] = (st[i].double() * (g1 - g0)).sum()
        return {"vol": _remap64(st, o, b, w), "grad_stack": gs, "grad_offsets": go}
    pc, ny = _affine_grid(c)
    vol = torch.empty((ny, r, k), dtype=torch.float64, device=DEV)
    z = torch.arange(k, device=DEV)
    pad = torch.zeros((1, r, k), dtype=torch.float32, device=DEV)
    st = torch.cat([pad, st.to(torch.int32).float(), pad, pad])      # images -1, N and N + 1
    for y in range(ny):
        u = (y * PIXEL - z.double() * pc) / c["step"]
        i = torch.floor(u)
        f = (u - i)[:, None]
        i = i.clamp(min=-2, max=n).long() + 1
        lo = torch.where((i >= 0)[:, None], st[i.clamp(min=0), :, z].double(), 0.0)
        vol[y] = ((1.0 - f) * lo + f * st[i + 1, :, z].double()).T
    return vol
