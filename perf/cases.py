"""The calls whose speed is measured, as a program that reconstructs the
corona makes them through paper_1103_5904_amd, and what each returns in 64
bits.

A case is a dict of plain values.  "kind" names the call; the rest describes
the cube (nx, ny, nz voxels on [-half, half]^3, frames), the views (layout,
nviews, ncol x nrow pixels, fov) and the options.  Lengths are in solar radii;
observers sit at 215 of them.  Layouts: "pairs", two observers at +-45 degrees
while the Sun turns 13.2 degrees a day, over 14 days; "ring", equally spaced
in longitude, starting 0.3 steps from 0 (no observer on an axis or a diagonal
of the cube: lines of sight along voxel faces belong to either side).
"""
from __future__ import annotations

import math
import os
from types import SimpleNamespace

import numpy as np
import torch

import paper_1103_5904_amd as tomo
from paper_1103_5904_amd import autograd as tomo_autograd
from paper_1103_5904_amd import precond as tomo_precond

R_OBS = 215.0
LAM_R, LAM_T = 1e-2, 10.0


def _case(name, kind, n, nviews, npix, *, layout="ring", half=1.5, fov=3.4, frames=1, map_mask=False,
          data_mask=False, obstacle=False, gains=False, iters=0, extras=False, brightness="pB"):
    c = {"kind": kind, "nx": n[0], "ny": n[1], "nz": n[2], "half": half, "frames": frames, "layout": layout,
         "nviews": nviews, "ncol": npix[0], "nrow": npix[1], "fov": fov, "map_mask": map_mask,
         "data_mask": data_mask, "obstacle": obstacle, "gains": gains, "iters": iters, "extras": extras,
         "brightness": brightness}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest model (32^3, 8 views of 32^2): a quick look, a unit
        # test, a loop of many small calls; launches and latency are its cost
        _case("project-tiny", "project", (32, 32, 32), 8, (32, 32), fov=3.2),
        _case("backproject-tiny", "backproject", (32, 32, 32), 8, (32, 32), fov=3.2),
        # the static EUVI-like model: two spacecraft, 14 days, pixels finer
        # than voxels, the Sun's interior masked out; each operator by itself
        # as a caller's own solver applies it
        _case("project-euvi", "project", (128, 128, 128), 28, (512, 512), layout="pairs", map_mask=True),
        _case("backproject-euvi", "backproject", (128, 128, 128), 28, (512, 512), layout="pairs", map_mask=True),
        # white light (COR1-like): polarised brightness of one large frame
        # under all 60 views, the coronagraph's annulus kept
        _case("thomson-cor1", "thomson", (256, 256, 256), 60, (512, 512), layout="pairs", half=4.0, fov=8.0,
              map_mask=True, data_mask=True),
        # images coarser than the cube: 64 views of 256^2 under 256^3, the
        # cube-size sweep's second point
        _case("project-sparse", "project", (256, 256, 256), 64, (256, 256), fov=3.2),
        # nothing round: an uneven cube, odd images, an opaque Sun, gains of
        # several instruments
        _case("backproject-ragged", "backproject", (193, 150, 77), 21, (301, 173), obstacle=True, gains=True),
        # gradient-based fitting: the criterion and its gradient through autograd
        _case("loss-step", "loss", (128, 128, 128), 32, (256, 256)),
        # a small inversion, a fixed number of iterations
        _case("cg-small", "cg", (64, 64, 64), 16, (256, 256), iters=20),
        # the learned preconditioner's inversion to a relative residual of 1e-3
        _case("fcg-learned", "fcg", (128, 128, 128), 28, (256, 256), layout="pairs", iters=200),
        # the time-dependent COR1-like model (8 frames, 60 views) solved
        # together with four smaller reconstructions, graph-captured iterations
        _case("batch-cor1", "batch", (256, 256, 256), 60, (512, 512), layout="pairs", half=4.0, fov=8.0, frames=8,
              map_mask=True, data_mask=True, iters=6, extras=True),
        # one training step of the preconditioner network: its output and the
        # gradient of its parameters for a given output gradient
        _case("train-128", "train", (128, 128, 128), 1, (1, 1)),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["project", "project", "project", "backproject", "backproject", "backproject", "thomson", "loss",
                       "loss", "cg", "cg", "fcg", "batch", "train", "train"])
    for _ in range(1000):
        top = {"loss": 160, "cg": 128, "fcg": 144, "batch": 144, "train": 144}.get(kind, 320)
        side = _log_int(rng, 24, top)
        n = tuple(max(8, int(side * rng.uniform(0.6, 1.4))) for _ in range(3))
        if rng.random() < 0.4:
            n = (max(8, side // 4 * 4),) * 3
        pix = _log_int(rng, 24, 512)
        layout = rng.choice(["ring", "pairs"])
        pix += pix % 2 if layout == "pairs" else 0  # no line of sight exactly along the diagonal
        npix = (pix, max(16, int(pix * rng.uniform(0.6, 1.0)))) if rng.random() < 0.5 else (pix, pix)
        frames = rng.randint(2, 6) if kind == "batch" else 1
        nviews = frames * 2 * rng.randint(1, 4) if kind == "batch" else _log_int(rng, 4, 64)
        white = kind == "thomson" or (kind in ("project", "backproject", "batch") and rng.random() < 0.3)
        half, fov = (4.0, 8.0) if white else (1.5, rng.choice([3.2, 3.4]))
        c = _case(None, kind, n, nviews, npix, layout=layout, half=half, fov=fov, frames=frames,
                  map_mask=kind not in ("loss", "fcg", "train") and rng.random() < 0.5,
                  data_mask=kind not in ("loss", "fcg", "train") and white and rng.random() < 0.7,
                  obstacle=kind in ("project", "backproject", "cg") and rng.random() < 0.2,
                  gains=kind in ("project", "backproject", "cg", "loss") and rng.random() < 0.2,
                  iters={"cg": rng.randint(5, 25), "fcg": 200, "batch": rng.randint(4, 10)}.get(kind, 0),
                  extras=kind == "batch" and rng.random() < 0.5, brightness=rng.choice(["pB", "B"]))
        if kind == "train":
            c.update(nviews=1, ncol=1, nrow=1, layout="ring", half=1.5, fov=3.4)
        if work(c)["flops"] <= _MOST.get(kind, 6e9):
            return c
    return c


# ------------------------------------------------------------ geometry


def _longitudes(layout, nviews):
    if layout == "ring":
        step = 360.0 / nviews
        return [step * (k + 0.3) for k in range(nviews)]
    steps = (nviews + 1) // 2
    return [(45.0, -45.0)[k % 2] - 13.2 * 14.0 * (k // 2) / max(1, steps) for k in range(nviews)]


def _views(layout, nviews, ncol, nrow, fov):
    rows = []
    for lon in np.deg2rad(_longitudes(layout, nviews)):
        obs = R_OBS * np.array([np.cos(lon), np.sin(lon), 0.0])
        w = -obs / R_OBS
        u = np.cross(w, [0.0, 0.0, 1.0])
        u = u / np.linalg.norm(u)
        cd = fov / (max(ncol, nrow) * R_OBS)
        rows.append(np.concatenate([obs, w, u, np.cross(u, w), [cd, cd], [(ncol - 1) / 2.0, (nrow - 1) / 2.0]]))
    return np.array(rows), np.tile(np.array([[ncol, nrow]], dtype=np.int32), (nviews, 1))


def _geometry(c):
    n, half = (c["nx"], c["ny"], c["nz"]), c["half"]
    views, npix = _views(c["layout"], c["nviews"], c["ncol"], c["nrow"], c["fov"])
    g = SimpleNamespace(n=n, lo=np.full(3, -half), hi=np.full(3, half), views=views, npix=npix, view_frame=None,
                        nframes=c["frames"], data_mask=None, map_mask=None, obstacle=None, gains=None)
    if c["frames"] > 1:  # two views per time step, the steps dealt to the frames in order
        steps = (c["nviews"] + 1) // 2
        g.view_frame = np.array([(k // 2) * c["frames"] // steps for k in range(c["nviews"])], dtype=np.int32)
    if c["map_mask"]:  # voxels inside the Sun are no unknowns
        x, y, z = np.meshgrid(*[-half + (np.arange(m) + 0.5) * 2 * half / m for m in n], indexing="ij")
        g.map_mask = (x * x + y * y + z * z >= 1.0).astype(np.uint8).transpose(2, 1, 0).copy()
    if c["data_mask"]:  # the coronagraph sees 1.4 to 4 solar radii
        cols = (np.arange(c["ncol"]) - views[0, 14]) * views[0, 12] * R_OBS
        rws = (np.arange(c["nrow"]) - views[0, 15]) * views[0, 13] * R_OBS
        rr = np.hypot(cols[None, :], rws[:, None])
        g.data_mask = np.tile(((rr >= 1.4) & (rr <= 4.0)).astype(np.uint8).ravel(), c["nviews"])
    if c["obstacle"]:
        g.obstacle = np.array([0.0, 0.0, 0.0, 1.0])
    if c["gains"]:
        g.gains = np.where(np.arange(c["nviews"]) % 2 == 0, 1.0, 1.27)
    return g


def _extra_cases(c):
    """The smaller reconstructions solved beside a batch's main system."""
    if not c["extras"]:
        return []
    out = []
    for num, den in ((1, 4), (3, 8), (1, 2), (3, 4)):
        n = tuple(max(8, m * num // den) for m in (c["nx"], c["ny"], c["nz"]))
        out.append(_case(None, "batch", n, 16, (max(16, c["ncol"] // 2), max(16, c["nrow"] // 2))))
    return out


# -------------------------------------------------------------- inputs


def _blobs(c, seed):
    """Sixteen Gaussian blobs of a corona: centre, width, amplitude."""
    r = np.random.default_rng(seed)
    s = c["half"] / 1.5
    return [(r.uniform(-1.2, 1.2, 3) * s, r.uniform(0.05, 0.3) * s, r.uniform(0.1, 1.0)) for _ in range(16)]


def _turned(mu, deg):
    a = math.radians(deg)
    return np.array([math.cos(a) * mu[0] - math.sin(a) * mu[1], math.sin(a) * mu[0] + math.cos(a) * mu[1], mu[2]])


def _cube(c, seed):
    """Blobs over a radial fall-off r^-8, frame f turned by half a degree each."""
    n, half = (c["nx"], c["ny"], c["nz"]), c["half"]
    ax = [-half + (torch.arange(m, device="cuda", dtype=torch.float64) + 0.5) * (2 * half / m) for m in n]
    r2 = ax[0][None, None, :] ** 2 + ax[1][None, :, None] ** 2 + ax[2][:, None, None] ** 2
    shell = torch.where(r2 >= 1.0, r2.clamp_min(1e-3) ** -4, torch.zeros_like(r2))
    out = torch.empty((c["frames"], n[2], n[1], n[0]), device="cuda", dtype=torch.float32)
    for f in range(c["frames"]):
        acc = shell.clone()
        for mu, sg, a in _blobs(c, seed):
            e = [torch.exp(-((ax[k] - m) ** 2) / (2 * sg * sg)) for k, m in enumerate(_turned(mu, 0.5 * f))]
            acc += (a * e[2])[:, None, None] * (e[1][:, None] * e[0][None, :])[None]
        out[f] = acc.float()
    return out if c["frames"] > 1 else out[0]


def _data(c, g, seed):
    """What the detectors see of the blobs (their line integrals in closed
    form) with 1% noise; masked pixels hold 0."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    blobs = _blobs(c, seed)
    out = []
    for k in range(c["nviews"]):
        v = torch.from_numpy(g.views[k]).cuda()
        x = (torch.arange(c["ncol"], device="cuda", dtype=torch.float64) - v[14]) * v[12]
        y = (torch.arange(c["nrow"], device="cuda", dtype=torch.float64) - v[15]) * v[13]
        d = v[3:6] + x[None, :, None] * v[6:9] + y[:, None, None] * v[9:12]
        dd = (d * d).sum(-1)
        frame = 0 if g.view_frame is None else int(g.view_frame[k])
        img = torch.zeros_like(dd)
        for mu, sg, a in blobs:
            m = torch.from_numpy(_turned(mu, 0.5 * frame)).cuda() - v[0:3]
            h2 = (m * m).sum() - (d @ m) ** 2 / dd
            img += a * sg * math.sqrt(2 * math.pi) * torch.exp(-h2 / (2 * sg * sg))
        out.append(img.reshape(-1))
    y = torch.cat(out)
    y = y + 0.01 * y.mean() * torch.randn(y.numel(), generator=gen, device="cuda", dtype=torch.float64)
    if g.data_mask is not None:
        y = y * torch.from_numpy(g.data_mask).cuda()
    return y.float()


def _weights(seed):
    """The shipped network, each weight off by a few per cent."""
    here = os.path.dirname(os.path.abspath(tomo.__file__))
    w = tomo_precond.load(os.path.join(here, "precond_weights.npz"))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return w * (1.0 + 0.03 * torch.randn(w.numel(), generator=gen, device="cuda"))


def _residual(c, seed):
    """A unit-norm residual-like volume: smooth structure plus noise."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = _cube(dict(c, frames=1), seed).double()
    x = x - x.mean()
    x = x + 0.1 * x.std() * torch.randn(x.shape, generator=gen, device="cuda", dtype=torch.float64)
    return (x / x.norm()).float()


def prepare(case, seed):
    c = case
    kind = c["kind"]
    if kind == "train":
        shape = (c["nz"], c["ny"], c["nx"])
        return {"case": c, "net": tomo.ConvNet(shape), "params": _weights(seed), "x": _residual(c, seed),
                "dout": _residual(c, seed + 1)}
    if kind == "batch":
        cs = [c] + _extra_cases(c)
        gs = [_geometry(k) for k in cs]
        dgs = [tomo.DeviceGeometry(g) for g in gs]
        ys = [_data(k, g, seed + i) for i, (k, g) in enumerate(zip(cs, gs))]
        return {"case": c, "batch": tomo.Batch(dgs), "ys": ys, "lam_t": [LAM_T] + [0.0] * (len(cs) - 1)}
    g = _geometry(c)
    s = {"case": c, "g": tomo.DeviceGeometry(g)}
    if kind in ("project", "thomson", "loss"):
        s["x"] = _cube(c, seed)
    if kind in ("backproject", "loss", "cg", "fcg"):
        s["y"] = _data(c, g, seed)
    if kind == "fcg":
        here = os.path.dirname(os.path.abspath(tomo.__file__))
        s["net"] = tomo_precond.load(os.path.join(here, "precond_weights.npz"))
    return s


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind == "project":
        return tomo.project(state["g"], state["x"])
    if kind == "backproject":
        return tomo.backproject(state["g"], state["y"])
    if kind == "thomson":
        return tomo.thomson_project(state["g"], state["x"], u=0.63, kind=c["brightness"])
    if kind == "loss":
        x = state["x"].detach().requires_grad_(True)
        loss = tomo_autograd.data_loss(x, state["g"], state["y"], LAM_R)
        loss.backward()
        return {"loss": loss.detach(), "grad": x.grad}
    if kind == "cg":
        return tomo.cg_solve(state["g"], state["y"], lam_r=LAM_R, max_iter=c["iters"])[0]
    if kind == "fcg":
        return tomo.cg_solve(state["g"], state["y"], lam_r=LAM_R, max_iter=c["iters"], rtol=1e-3, check_every=5,
                             precond=state["net"])[0]
    if kind == "batch":
        return state["batch"].cg_solve(state["ys"], lam_r=LAM_R, lam_t=state["lam_t"], max_iter=c["iters"],
                                       check_every=c["iters"], use_graph=True)[0]
    z = state["net"].forward(state["params"], state["x"])
    return {"out": z, "grad": state["net"].backward(state["params"], state["x"], state["dout"])}


# ---------------------------------------------------------------- work


def _crossings(c):
    """Voxels crossed by all kept lines of sight, from a sample of each
    view's: one per plane crossed, and one."""
    views, _ = _views(c["layout"], c["nviews"], c["ncol"], c["nrow"], c["fov"])
    some = views[:: max(1, c["nviews"] // 8)]
    fx = np.linspace(0, c["ncol"] - 1, min(24, c["ncol"]))
    fy = np.linspace(0, c["nrow"] - 1, min(24, c["nrow"]))
    tot = 0.0
    for v in some:
        x, y = (fx - v[14]) * v[12], (fy - v[15]) * v[13]
        d = v[3:6] + x[None, :, None] * v[6:9] + y[:, None, None] * v[9:12]
        inv = 1.0 / np.where(d == 0, 1e-300, d)
        t1, t2 = (-c["half"] - v[0:3]) * inv, (c["half"] - v[0:3]) * inv
        lo, hi = np.minimum(t1, t2).max(-1), np.maximum(t1, t2).min(-1)
        n = np.array([c["nx"], c["ny"], c["nz"]])
        steps = (np.abs(d) * (hi - lo)[..., None] * n / (2 * c["half"])).sum(-1) + 1.0
        steps = np.where(hi > lo, steps, 0.0)
        if c["data_mask"]:
            rr = np.hypot(x[None, :], y[:, None]) * R_OBS
            steps = np.where((rr >= 1.4) & (rr <= 4.0), steps, 0.0)
        tot += steps.mean()
    return tot / len(some) * c["nviews"] * c["ncol"] * c["nrow"]


def work(case):
    """One multiply and add per voxel crossed and application of P or P^T (27
    taps per channel pair for the network); every input read once, every
    output written once."""
    c = case
    vox = float(c["nx"]) * c["ny"] * c["nz"] * c["frames"]
    if c["kind"] == "train":
        macs = 27.0 * (16 + 256 + 16)
        return {"bytes": 4.0 * (3 * vox + 2 * tomo.NPARAMS), "flops": 2.0 * vox * (3 * macs - 27 * 16)}
    pix = float(c["nviews"]) * c["ncol"] * c["nrow"]
    masks = (vox / c["frames"] if c["map_mask"] else 0.0) + (pix if c["data_mask"] else 0.0)
    one = 2.0 * _crossings(c)
    bytes_, flops = 4.0 * (vox + pix) + masks, one
    if c["kind"] == "loss":
        bytes_, flops = 4.0 * (2 * vox + pix), 2 * one + 16.0 * vox
    elif c["kind"] == "thomson":
        flops = one * (2 if c["brightness"] == "B" else 1) + 60.0 * vox
    elif c["kind"] in ("cg", "fcg", "batch"):
        its = 16 if c["kind"] == "fcg" else c["iters"]
        flops = one * (2 * its + 3) + 25.0 * vox * its
        if c["kind"] == "fcg":
            flops += 2.0 * vox * its * 27.0 * (16 + 256 + 16)
        for e in _extra_cases(c):
            w = work(dict(e, iters=c["iters"]))
            bytes_, flops = bytes_ + w["bytes"], flops + w["flops"]
    return {"bytes": bytes_, "flops": flops}


# the most work of a drawn case, by kind: below the largest listed one's time
_MOST = {"cg": 3e10, "batch": 6e10, "fcg": 4e11, "train": 1.2e11}


# --------------------------------------------------------------- exact


def _segments(g, k, keep=None, limit=8_000_000):
    """Chunks (pixels, voxels [rays, 3 slabs], lengths) of view k's lines of
    sight: along a ray's steepest axis each slab of voxels is crossed once, and
    in it at most one plane of each other axis, so three pieces cover it."""
    f8 = dict(device="cuda", dtype=torch.float64)
    v = torch.tensor(g.views[k], **f8)
    ncol, nrow = (int(m) for m in g.npix[k])
    n = torch.tensor(g.n, **f8)
    lo, hi = torch.tensor(g.lo, **f8), torch.tensor(g.hi, **f8)
    delta = (hi - lo) / n
    x = (torch.arange(ncol, **f8) - v[14]) * v[12]
    y = (torch.arange(nrow, **f8) - v[15]) * v[13]
    d = (v[3:6] + x[None, :, None] * v[6:9] + y[:, None, None] * v[9:12]).reshape(-1, 3)
    o = v[0:3]
    inv = 1.0 / torch.where(d == 0, torch.full_like(d, 1e-300), d)
    t1, t2 = (lo - o) * inv, (hi - o) * inv
    tin = torch.minimum(t1, t2).amax(1).clamp_min(0.0)
    tout = torch.maximum(t1, t2).amin(1)
    if g.obstacle is not None:
        oc = o - torch.tensor(g.obstacle[:3], **f8)
        dd, od = (d * d).sum(1), d @ oc
        ts = -od / dd
        h2 = ((oc + ts[:, None] * d) ** 2).sum(1)
        r2 = float(g.obstacle[3]) ** 2
        tc = ts - ((r2 - h2).clamp_min(0.0) / dd).sqrt()
        tout = torch.where((h2 < r2) & (ts > 0), torch.minimum(tout, tc), tout)
    ok = tout > tin
    if keep is not None:
        ok = ok & keep
    e = d / delta
    p = (o - lo) / delta
    major = e.abs().argmax(1)
    norm = d.norm(dim=1)
    for a in range(3):
        rays = torch.nonzero(ok & (major == a)).reshape(-1)
        if not rays.numel():
            continue
        b, c = [q for q in range(3) if q != a]
        na = int(g.n[a])
        slab = torch.arange(na, **f8)
        for r in torch.split(rays, max(1, limit // na)):
            ea, eb, ec = (e[r, q][:, None] for q in (a, b, c))
            ta, tb = (slab[None, :] - p[a]) / ea, (slab[None, :] + 1.0 - p[a]) / ea
            s0, s1 = tin[r][:, None], tout[r][:, None]
            t0 = torch.minimum(torch.maximum(torch.minimum(ta, tb), s0), s1)
            tz = torch.minimum(torch.maximum(torch.maximum(ta, tb), s0), s1)
            cut = []
            for q, eq in ((b, eb), (c, ec)):
                plane = torch.floor(torch.maximum(p[q] + eq * t0, p[q] + eq * tz))
                t = (plane - p[q]) / eq
                cut.append(torch.minimum(torch.maximum(torch.where(eq == 0, tz, t), t0), tz))
            ends = [t0, torch.minimum(*cut), torch.maximum(*cut), tz]
            idx, length = [], []
            for i in range(3):
                mid = 0.5 * (ends[i] + ends[i + 1])
                co = [None] * 3
                for q, eq in ((a, ea), (b, eb), (c, ec)):
                    co[q] = (p[q] + eq * mid).floor().clamp(0, int(g.n[q]) - 1).long()
                idx.append((co[2] * int(g.n[1]) + co[1]) * int(g.n[0]) + co[0])
                length.append((ends[i + 1] - ends[i]) * norm[r][:, None])
            yield r, torch.cat(idx, 1), torch.cat(length, 1)


def _each_segment(g):
    pix = g.npix[:, 0].astype(np.int64) * g.npix[:, 1]
    off = np.concatenate([[0], np.cumsum(pix)])
    for k in range(len(pix)):
        keep = None
        if g.data_mask is not None:
            keep = torch.from_numpy(g.data_mask[off[k]:off[k + 1]]).cuda() != 0
        gain = 1.0 if g.gains is None else float(g.gains[k])
        for r, idx, length in _segments(g, k, keep):
            yield r + int(off[k]), idx, length * gain


def _map(g):
    return None if g.map_mask is None else torch.from_numpy(g.map_mask).cuda().reshape(-1).double()


def _project64(g, x, segs=None):
    npix = int((g.npix[:, 0].astype(np.int64) * g.npix[:, 1]).sum())
    m = _map(g)
    x = x.reshape(-1).double()
    x = x if m is None else x * m
    out = torch.zeros(npix, device="cuda", dtype=torch.float64)
    for pix, idx, length in segs or _each_segment(g):
        out[pix] = (x[idx] * length).sum(1)
    return out


def _backproject64(g, y, segs=None):
    y = y.double()
    out = torch.zeros(int(np.prod(g.n)), device="cuda", dtype=torch.float64)
    for pix, idx, length in segs or _each_segment(g):
        w = (length * y[pix][:, None]).reshape(-1)
        some = torch.nonzero(w).reshape(-1)
        out.index_add_(0, idx.reshape(-1)[some], w[some])
    m = _map(g)
    return out if m is None else out * m


def _prior64(shape, x):
    x = x.reshape(shape)
    out = torch.zeros_like(x)
    for a in range(3):
        n = shape[a]
        if n > 1:
            d = x.narrow(a, 1, n - 1) - x.narrow(a, 0, n - 1)
            out.narrow(a, 1, n - 1).add_(d)
            out.narrow(a, 0, n - 1).sub_(d)
    return out.reshape(-1)


def _thomson64(c, g, x):
    half, n = c["half"], g.n
    ax = [-half + (torch.arange(m, device="cuda", dtype=torch.float64) + 0.5) * (2 * half / m) for m in n]
    r = (ax[0][None, None, :] ** 2 + ax[1][None, :, None] ** 2 + ax[2][:, None, None] ** 2).sqrt().reshape(-1)
    u, out = 0.63, r > 1.0
    rr = torch.where(out, r, torch.full_like(r, 2.0))
    s = 1.0 / rr
    co = (1.0 - s * s).sqrt()
    lg = torch.log((1.0 + s) / co) * co * co / s
    c1, c2 = co * s * s, -(1.0 - 3.0 * s * s - lg * (1.0 + 3.0 * s * s)) / 8.0
    c3, c4 = 4.0 / 3.0 - co - co ** 3 / 3.0, (5.0 + s * s - lg * (5.0 - s * s)) / 8.0
    zero = torch.zeros_like(r)
    m = torch.where(out, ((1 - u) * c1 + u * c2) / rr ** 4, zero)
    mp = torch.where(out, 2.0 * ((1 - u) * c3 + u * c4) / rr ** 2, zero)
    x = x.reshape(-1).double()
    rho2 = []
    for v in torch.from_numpy(g.views).cuda():
        px = (torch.arange(c["ncol"], device="cuda", dtype=torch.float64) - v[14]) * v[12]
        py = (torch.arange(c["nrow"], device="cuda", dtype=torch.float64) - v[15]) * v[13]
        d = (v[3:6] + px[None, :, None] * v[6:9] + py[:, None, None] * v[9:12]).reshape(-1, 3)
        cr = torch.linalg.cross(v[0:3].expand_as(d), d)
        rho2.append((cr * cr).sum(1) / (d * d).sum(1))
    rho2 = torch.cat(rho2)
    img = rho2 * _project64(g, m * x)
    return img if c["brightness"] == "pB" else _project64(g, mp * x) - img


def _conv64(x, w, b):
    """3x3x3 zero-padded correlation, channels first, as 27 matrix products."""
    nz, ny, nx = x.shape[1:]
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1, 1, 1))
    out = b[:, None].expand(-1, nz * ny * nx)
    for t in range(27):
        dz, dy, dx = t // 9, (t // 3) % 3, t % 3
        out = out + w[:, :, t] @ xp[:, dz:dz + nz, dy:dy + ny, dx:dx + nx].reshape(x.shape[0], -1)
    return out.reshape(-1, nz, ny, nx)


def _network64(params, x):
    p = params
    w1, b1 = p[0:432].reshape(16, 1, 27), p[432:448]
    w2, b2 = p[448:7360].reshape(16, 16, 27), p[7360:7376]
    w3, b3 = p[7376:7808].reshape(1, 16, 27), p[7808:7809]
    a = torch.relu(_conv64(x[None], w1, b1))
    return _conv64(torch.relu(_conv64(a, w2, b2)), w3, b3)[0]


def _cg64(c, g, y):
    """The textbook recurrence, from zero, a fixed number of iterations."""
    segs = list(_each_segment(g))
    shape = (c["nz"], c["ny"], c["nx"])
    m = _map(g)

    def apply(v):
        q = _backproject64(g, _project64(g, v, segs), segs)
        pr = LAM_R * _prior64(shape, v)
        return q + (pr if m is None else pr * m)

    r = _backproject64(g, y, segs)
    x, p = torch.zeros_like(r), r.clone()
    rr = r @ r
    for _ in range(c["iters"]):
        q = apply(p)
        alpha = rr / (p @ q)
        x, r = x + alpha * p, r - alpha * q
        new = r @ r
        p = r + (new / rr) * p
        rr = new
    return x


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind in ("fcg", "batch"):  # hundreds of applications, or a network that rounds to 16 bits inside
        return None
    if kind == "train":
        params = _weights(seed).double().requires_grad_(True)
        z = _network64(params, _residual(c, seed).double())
        z.backward(_residual(c, seed + 1).double())
        return {"out": z.detach(), "grad": params.grad}
    g = _geometry(c)
    shape = (c["nz"], c["ny"], c["nx"])
    if kind == "project":
        return _project64(g, _cube(c, seed))
    if kind == "backproject":
        return _backproject64(g, _data(c, g, seed)).reshape(shape)
    if kind == "thomson":
        return _thomson64(c, g, _cube(c, seed))
    if kind == "cg":
        # the segments are kept for all iterations: 20 bytes each
        if _crossings(c) * 3 * 20 > 6e10:
            return None
        return _cg64(c, g, _data(c, g, seed)).reshape(shape)
    x, y = _cube(c, seed).double().reshape(-1), _data(c, g, seed).double()
    r = _project64(g, x) - y
    lx = LAM_R * _prior64(shape, x)
    grad = _backproject64(g, r) + 2.0 * lx
    return {"loss": 0.5 * (r @ r) + x @ lx, "grad": grad.reshape(shape)}
