"""Performance cases: the calls a user of the beamformer makes, with the sizes
they are made at.

A case is a dict of plain values; ``kind`` names the call:

  frame    Plan.beamform: one frame at one order, one launch
  orders   Plan.beamform_orders: orders 1..max_order of one frame in one pass
  batch    Batch.launch: the frames of one plan in one persistent launch per
           order order_lo..order_hi
  mixed    Batch.replay: frames of several plans and orders in one graph
  serve    Batch.set + Batch.launch: a serving loop's submission, whose list
           of requests is new on each pass
  display  Display.run (images = 1) or Display.run_batch: band-pass, envelope
           and dB image of beamformed images
  metrics  image_metrics: SNR, CR, gCNR and FWHM of an envelope image

The array, field of view and phantom follow the package's own workloads: pitch
0.3 mm, 1540 m/s, 40 MHz, an image as wide as the array and as deep as the
record; point and line absorbers with a 5 MHz pulse in channel noise.
"""
import math
import random

import numpy as np
import torch

from paper_2203_14906_amd import hodmas
from paper_2203_14906_amd.phantom import Geometry, Grid

C, FS, PITCH, F0 = 1540.0, 40e6, 0.3e-3, 5e6
ADC = 8191                      # 14-bit signed codes
TAPS, BAND, RANGE_DB = 63, (2e6, 8e6), 60.0
DEV = "cuda"


# ---------------------------------------------------------------- the cases
def frame(name, n, s, nx, nz, dtype, order, mirror=False, cf=False, t0_us=0.0, given=False):
    c = {"kind": "frame", "n": n, "s": s, "nx": nx, "nz": nz, "dtype": dtype, "order": order, "mirror": mirror,
         "cf": cf, "t0_us": t0_us, "given": given}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest frame the package benchmarks, as a live display forms
        # it: a launch of a few microseconds, where latency is everything
        frame("frame_128_f32_k2", 64, 1024, 128, 128, "f32", 2),
        # the usual frame at the paper's DMAS-3, general array (no pairing)
        frame("frame_512_f32_k3", 128, 2048, 512, 512, "f32", 3),
        # raw ADC codes of a large array at the highest order
        frame("frame_1024_i16_k6", 256, 2048, 1024, 1024, "i16", 6),
        # the largest image of the paper's timing table, symmetric array
        frame("frame_2048_f32_k5_mirror", 128, 2048, 2048, 2048, "f32", 5, mirror=True),
        # a calibrated array (measured positions), a record that starts after
        # the shot, an image of no round size, coherence weighting
        frame("frame_331x203_f16_k4_cf", 96, 1500, 331, 203, "f16", 4, cf=True, t0_us=2.5, given=True),
        # the comparison of DAS, DMAS and DMAS-3..6 on one frame
        {"name": "orders_512_f32", "kind": "orders", "n": 128, "s": 2048, "nx": 512, "nz": 512, "dtype": "f32",
         "max_order": 6},
        # a cine of 8 resident frames at every order (the benchmark's step)
        {"name": "batch_8x512_f32_mirror", "kind": "batch", "frames": 8, "n": 128, "s": 2048, "nx": 512, "nz": 512,
         "dtype": "f32", "order_lo": 1, "order_hi": 6, "mirror": True},
        # reprocessing: frames of several arrays, depths and sizes in one graph
        {"name": "mixed_24_f16", "kind": "mixed", "frames": 24, "mix": 4000, "dtype": "f16", "mirror": True},
        # one submission of a loaded frame server
        {"name": "serve_16_f16", "kind": "serve", "frames": 16, "mix": 5000, "dtype": "f16", "mirror": True},
        # the display of one live image
        {"name": "display_512", "kind": "display", "images": 1, "nx": 512, "nz": 512, "envelope": True},
        # the display of a stored cine
        {"name": "display_16x1024", "kind": "display", "images": 16, "nx": 1024, "nz": 1024, "envelope": False},
        # quality of a large image: a lesion against the tissue around it
        {"name": "metrics_1024", "kind": "metrics", "nx": 1024, "nz": 1024, "target": 160, "background": 400,
         "bins": 256},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    most = 2048 * 2048 * 128    # pixel-channels of the largest listed frame
    kind = rng.choice(["frame"] * 6 + ["orders", "batch", "batch", "mixed", "serve", "display", "display", "metrics"])
    dtype = rng.choice(["f32", "f16", "i16"])
    n, s = _log(rng, 16, 256), _log(rng, 512, 4096)
    if kind in ("mixed", "serve"):
        return {"kind": kind, "frames": _log(rng, 2, 24 if kind == "mixed" else 16), "mix": rng.randrange(1 << 20),
                "dtype": rng.choice(["f16", "f32"]), "mirror": rng.random() < 0.7}
    if kind == "display":
        nz = 1 << rng.randrange(7, 12)
        nx = _log(rng, 64, 1024)
        return {"kind": kind, "images": _log(rng, 1, max(1, min(16, (16 << 20) // (nx * nz)))), "nx": nx, "nz": nz,
                "envelope": rng.random() < 0.5}
    if kind == "metrics":
        nx, nz = _log(rng, 128, 1024), _log(rng, 128, 1024)
        side = min(nx, nz)
        return {"kind": kind, "nx": nx, "nz": nz, "target": _log(rng, 8, side // 3),
                "background": _log(rng, 16, side // 2), "bins": rng.choice([64, 100, 256])}
    if kind == "orders":
        nx, nz = _log(rng, 64, 640), _log(rng, 64, 640)
        return {"kind": kind, "n": n, "s": s, "nx": nx, "nz": nz, "dtype": dtype, "max_order": rng.randrange(2, 7)}
    if kind == "batch":
        mirror = rng.random() < 0.5
        nx, nz = _log(rng, 64, 512), _log(rng, 64, 512)
        lo = rng.randrange(1, 7)
        return {"kind": kind, "frames": _log(rng, 2, 8), "n": min(n, 128), "s": s,
                "nx": (nx + 15) // 16 * 16 if mirror else nx, "nz": nz, "dtype": dtype, "order_lo": lo,
                "order_hi": rng.randrange(lo, 7), "mirror": mirror}
    nx, nz = _log(rng, 64, 2048), _log(rng, 64, 2048)
    while nx * nz * n > most:
        nx, nz = max(64, nx * 3 // 4), max(64, nz * 3 // 4)
    if rng.random() < 0.25:     # four pixel columns per element, as the usual frame has
        nx, nz = 4 * n, min(nz, most // (4 * n * n))
    given = rng.random() < 0.2
    mirror = not given and rng.random() < 0.4
    return frame(None, n, s, max(16, nx // 16 * 16) if mirror else nx, nz, dtype, rng.randrange(1, 7), mirror=mirror,
                 cf=rng.random() < 0.2, t0_us=round(rng.uniform(0.5, 4.0), 2) if rng.random() < 0.3 else 0.0,
                 given=given)


# ---------------------------------------------------------------- the inputs
def _element_x(case, seed):
    """Element positions: centred and uniform, or (given) each off by up to 10
    % of the pitch, as a calibration measures them."""
    n = case["n"]
    x = (np.arange(n) - (n - 1) / 2.0) * PITCH
    if case.get("given"):
        x = x + np.random.default_rng(seed).uniform(-0.1, 0.1, n) * PITCH
    return x


def _grid(n, s, nx, nz):
    width, depth = n * PITCH, 20e-3 * s / 1024.0
    dx, dz = width / nx, depth / nz
    return Grid(nx=nx, nz=nz, x0_m=-width / 2.0 + dx / 2.0, dx_m=dx, z0_m=dz / 2.0, dz_m=dz)


def _record(n, s, t0, xe, seed):
    """float64 [n][s] on the GPU: 40 point absorbers and 2 lines, each a
    Gaussian-derivative pulse that falls off as 1/r, in channel noise; the
    largest sample is 1.  Formed source by source, so the sums do not depend
    on the order of any atomics."""
    g = np.random.default_rng(seed)
    width, depth = n * PITCH, 20e-3 * s / 1024.0
    src = [(g.uniform(-width / 2, width / 2), g.uniform(1e-3, depth), g.uniform(0.5, 1.0)) for _ in range(40)]
    for _ in range(2):
        cx, cz, ang, amp = g.uniform(-width / 2, width / 2), g.uniform(4e-3, depth), g.uniform(0, math.pi), g.uniform(
            0.3, 0.8)
        for a in np.linspace(-4e-3, 4e-3, 24):
            x, z = cx + a * math.cos(ang), cz + a * math.sin(ang)
            if z > 0.5e-3:
                src.append((x, z, amp / 4))
    xd = torch.from_numpy(xe).to(DEV)
    t = torch.arange(s, dtype=torch.float64, device=DEV) / FS + t0
    rf = torch.zeros((n, s), dtype=torch.float64, device=DEV)
    sigma = 1.0 / (2.0 * math.pi * F0)
    for x, z, a in src:
        r = torch.sqrt((x - xd) ** 2 + z * z)
        u = (t[None, :] - (r / C)[:, None]) / sigma
        rf -= (a / (r * 1e3))[:, None] * u * torch.exp(-0.5 * u * u)
    rms = rf.square().mean(dim=1, keepdim=True).sqrt()
    rms = torch.where(rms > 0, rms, rms.max())
    noise = torch.from_numpy(g.standard_normal((n, s))).to(DEV)
    rf = rf + noise * rms * 10.0 ** (-15.0 / 20.0)
    return rf / rf.abs().max()


def _store(rf, dtype, seed):
    """(stored record, the value of one code)."""
    if dtype == "f32":
        return rf.float(), 1.0
    if dtype == "f16":
        return rf.half(), 1.0
    u = np.random.default_rng(seed ^ 0x5EED).uniform(0.5, 0.95)
    return torch.clamp(torch.round(rf * (u * ADC)), -ADC, ADC).to(torch.int16), float(np.float32(1.0 / (u * ADC)))


def _frame_inputs(case, seed, k=0):
    """(positions, t0, stored record, scale) of the case's k-th frame."""
    xe = _element_x(case, seed)
    t0 = case.get("t0_us", 0.0) * 1e-6
    rf = _record(case["n"], case["s"], t0, xe, seed * 64 + k)
    stored, scale = _store(rf, case["dtype"], seed * 64 + k)
    return xe, t0, stored, scale


def _plan(case, xe, t0, scale, order, flags=0):
    geom = Geometry(case["n"], t0_s=t0, element_x_m=xe if case.get("given") else None)
    return hodmas.Plan(geom, _grid(case["n"], case["s"], case["nx"], case["nz"]), case["s"], case["dtype"],
                       max_order=order, dequant_scale=scale, frame_max=1.0 if case["dtype"] == "i16" else 0.0,
                       flags=flags)


def _image(nx, nz):
    return torch.zeros((nz, nx), dtype=torch.float32, device=DEV)


def _members(case):
    """The frames of a mixed batch: shapes and orders from the case's mix."""
    r = random.Random(case["mix"])
    out = []
    for _ in range(case["frames"]):
        side = r.choice([256, 512, 768] if case["kind"] == "mixed" else [256, 512])
        out.append({"n": r.choice([64, 128, 256]), "s": r.choice([1024, 2048, 4096]), "nx": side, "nz": side,
                    "dtype": case["dtype"], "order": r.randrange(1, 7)})
    return out


def _envelope_image(case, seed):
    """A speckle image with a bright target, as the envelope of a beamformed
    image has it, and its two rectangles."""
    nx, nz, side, back = case["nx"], case["nz"], case["target"], case["background"]
    g = np.random.default_rng(seed)
    im = g.rayleigh(1.0, (nz, nx))
    tx, tz = int(g.integers(0, nx - side + 1)), int(g.integers(0, nz - side + 1))
    x, z = np.arange(nx) - tx - side / 2.0, np.arange(nz) - tz - side / 2.0
    im += 12.0 * np.exp(-(x[None, :] ** 2 + z[:, None] ** 2) / (2.0 * (side / 4.0) ** 2))
    bx, bz = int(g.integers(0, nx - back + 1)), int(g.integers(0, nz - back + 1))
    return im.astype(np.float32), (tx, tx + side, tz, tz + side), (bx, bx + back, bz, bz + back)


def _beam_images(case, seed):
    """Beamformed images to display: band-limited echoes along depth in
    noise, brighter in places."""
    nx, nz = case["nx"], case["nz"]
    g = torch.Generator().manual_seed(seed)
    fs = C / (20e-3 / nz * 2)
    z = torch.arange(nz, dtype=torch.float32)[:, None]
    out = []
    for _ in range(case["images"]):
        amp = torch.rand((1, nx), generator=g) ** 4 * torch.exp(-((z - nz * torch.rand((1, nx), generator=g)) / 20) ** 2)
        ph = 6.28 * torch.rand((1, nx), generator=g)
        im = amp * torch.cos(2 * math.pi * F0 / fs * z + ph) + 0.01 * torch.randn((nz, nx), generator=g)
        out.append(im.to(DEV).contiguous())
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("frame", "orders"):
        order = case.get("order") or case["max_order"]
        flags = (hodmas.FLAG_MIRROR if case.get("mirror") else 0) | (hodmas.FLAG_CF if case.get("cf") else 0)
        xe, t0, rf, scale = _frame_inputs(case, seed)
        images = [_image(case["nx"], case["nz"]) for _ in range(order if kind == "orders" else 1)]
        return {"kind": kind, "plan": _plan(case, xe, t0, scale, order, flags), "rf": rf, "order": order,
                "out": images if kind == "orders" else images[0]}
    if kind == "batch":
        flags = hodmas.FLAG_MIRROR if case["mirror"] else 0
        ins = [_frame_inputs(case, seed, k) for k in range(case["frames"])]
        # int16 frames have a scale, hence a plan, each
        scales = sorted({i[3] for i in ins})
        plans = {s: _plan(case, ins[0][0], 0.0, s, case["order_hi"], flags) for s in scales}
        rfs, per = [i[2] for i in ins], [plans[i[3]] for i in ins]
        info = per[0].info()
        batches, outs = [], []
        for k in range(case["order_lo"], case["order_hi"] + 1):
            images = [_image(case["nx"], case["nz"]) for _ in rfs]
            b = hodmas.Batch(len(rfs), len(rfs) * info.n_tiles, info.lds_bytes)
            b.set(per, rfs, [k] * len(rfs), images)
            batches.append(b)
            outs.append(images)
        return {"kind": kind, "batches": batches, "out": outs}
    if kind in ("mixed", "serve"):
        flags = hodmas.FLAG_MIRROR if case["mirror"] else 0
        plans, records, use, rfs, orders, images = {}, {}, [], [], [], []
        for m in _members(case):
            rec, shape = (m["n"], m["s"]), (m["n"], m["s"], m["nx"])
            if rec not in records:
                records[rec] = _frame_inputs(m, seed)
            if shape not in plans:
                plans[shape] = _plan(m, records[rec][0], 0.0, 1.0, 6, flags)
            use.append(plans[shape])
            rfs.append(records[rec][2])
            orders.append(m["order"])
            images.append(_image(m["nx"], m["nz"]))
        infos = [p.info() for p in use]
        b = hodmas.Batch(len(use), sum(i.n_tiles for i in infos), max(i.lds_bytes for i in infos))
        st = {"kind": kind, "batch": b, "plans": use, "rfs": rfs, "orders": orders, "out": images}
        if kind == "mixed":
            b.set(use, rfs, orders, images)
            b.capture()
        return st
    if kind == "display":
        ims = _beam_images(case, seed)
        d = hodmas.Display(case["nx"], case["nz"], 40e-3 / case["nz"], C, *_band(case), numtaps=TAPS,
                           dynamic_range_db=RANGE_DB)
        return {"kind": kind, "display": d, "images": ims,
                "env": [_image(case["nx"], case["nz"]) for _ in ims] if case["envelope"] else None,
                "db": [_image(case["nx"], case["nz"]) for _ in ims]}
    im, target, background = _envelope_image(case, seed)
    return {"kind": kind, "image": torch.from_numpy(im).to(DEV), "dx": PITCH / 4, "target": target,
            "background": background, "bins": case["bins"]}


def run(state):
    kind = state["kind"]
    if kind == "frame":
        return state["plan"].beamform(state["rf"], state["order"], state["out"])
    if kind == "orders":
        return state["plan"].beamform_orders(state["rf"], state["order"], state["out"])
    if kind == "batch":
        for b in state["batches"]:
            b.launch()
        return state["out"]
    if kind == "mixed":
        state["batch"].replay()
        return state["out"]
    if kind == "serve":
        state["batch"].set(state["plans"], state["rfs"], state["orders"], state["out"])
        state["batch"].launch()
        return state["out"]
    if kind == "display":
        if len(state["images"]) == 1:
            env, db = state["display"].run(state["images"][0], state["env"][0] if state["env"] else None, state["db"][0])
            return [db] if env is None else [env, db]
        env, db = state["display"].run_batch(state["images"], state["env"], state["db"])
        return db if env is None else [*env, *db]
    return hodmas.image_metrics(state["image"], state["dx"], state["target"], state["background"], state["bins"])


# ------------------------------------------------------------------ the work
def _frame_work(c, orders):
    """Record(s) once, one image per order; per pixel and channel about ten
    operations for the delay and the interpolation's place, three for the
    interpolation, two for a root, and 2k for the sums of order k."""
    size = 4 if c["dtype"] == "f32" else 2
    pix = c["nx"] * c["nz"]
    return {"bytes": c["n"] * c["s"] * size + 4 * pix * len(orders),
            "flops": pix * c["n"] * (13 + sum(2 * k + (2 if k > 1 else 0) for k in orders))}


def work(case):
    kind = case["kind"]
    if kind == "frame":
        return _frame_work(case, [case["order"]])
    if kind == "orders":
        return _frame_work(case, range(1, case["max_order"] + 1))
    if kind in ("batch", "mixed", "serve"):
        parts = ([_frame_work(case, [k]) for k in range(case["order_lo"], case["order_hi"] + 1)] * case["frames"]
                 if kind == "batch" else [_frame_work(m, [m["order"]]) for m in _members(case)])
        return {"bytes": sum(p["bytes"] for p in parts), "flops": sum(p["flops"] for p in parts)}
    pix = case["nx"] * case["nz"]
    if kind == "display":       # image in, dB image (and envelope) out; FIR and two FFTs along depth
        each = pix * (2 * TAPS + 10 * math.log2(case["nz"]) + 10)
        return {"bytes": 4 * pix * (3 if case["envelope"] else 2) * case["images"], "flops": each * case["images"]}
    pix = case["target"] ** 2 + case["background"] ** 2
    return {"bytes": 4 * pix, "flops": 8 * pix}


# --------------------------------------------------- the same in 64 bits
def _exact_frames(c, xe, t0, stored, scale, orders, cf=False):
    """Images of the stored records (one geometry) at the orders, in float64:
    [record][order] -> tensor [nz][nx]."""
    g = _grid(c["n"], c["s"], c["nx"], c["nz"])
    n, s = c["n"], c["s"]
    px = (g.x0_m + torch.arange(c["nx"], dtype=torch.float64, device=DEV) * g.dx_m)[None, :]
    pz = (g.z0_m + torch.arange(c["nz"], dtype=torch.float64, device=DEV) * g.dz_m)[:, None]
    recs = [r.double() * sc for r, sc in zip(stored, scale)]
    E = [[[torch.zeros((c["nz"], c["nx"]), dtype=torch.float64, device=DEV) for _ in range(k)] for k in orders]
         for _ in recs]
    s1 = [torch.zeros((c["nz"], c["nx"]), dtype=torch.float64, device=DEV) for _ in recs]
    s2 = [torch.zeros_like(a) for a in s1]
    for i in range(n):
        t = FS * (torch.sqrt((px - xe[i]) ** 2 + pz * pz) / C - t0)
        ok = (t >= 0) & (t <= s - 1)
        j = torch.clamp(t.floor().long(), 0, s - 2)
        f = torch.where(ok, t - j, torch.zeros_like(t))
        for r, rec in enumerate(recs):
            v = torch.where(ok, (1 - f) * rec[i][j] + f * rec[i][j + 1], torch.zeros_like(f))
            if cf:
                s1[r] += v
                s2[r] += v * v
            for o, k in enumerate(orders):
                y = v if k == 1 else torch.sign(v) * v.abs() ** (1.0 / k)
                e = E[r][o]
                for m in range(k - 1, 0, -1):
                    e[m] += y * e[m - 1]
                e[0] += y
    out = [[E[r][o][-1] for o in range(len(list(orders)))] for r in range(len(recs))]
    if cf:
        for r in range(len(recs)):
            w = torch.where(s2[r] > 0, s1[r] ** 2 / (n * s2[r]), torch.zeros_like(s1[r]))
            out[r] = [w * e for e in out[r]]
    return out


def _band(case):
    """The pass band, inside what the image's depth sampling carries."""
    half = 0.5 * C / (40e-3 / case["nz"])
    return (min(BAND[0], 0.2 * half), min(BAND[1], 0.8 * half))


def _taps(case):
    fs = C / (40e-3 / case["nz"])
    lo, hi = (f / fs for f in _band(case))
    m = np.arange(TAPS) - (TAPS - 1) / 2
    h = 2 * hi * np.sinc(2 * hi * m) - 2 * lo * np.sinc(2 * lo * m)
    h *= 0.54 - 0.46 * np.cos(2 * np.pi * np.arange(TAPS) / (TAPS - 1))
    return h / np.sum(h * np.cos(np.pi * (lo + hi) * m))


def _exact_display(im, taps):
    nz, nx = im.shape
    half = (TAPS - 1) // 2
    pad = torch.zeros((nz + 2 * half, nx), dtype=torch.float64, device=DEV)
    pad[half:half + nz] = im.double()
    x = sum(float(taps[k]) * pad[k:k + nz] for k in range(TAPS))
    X = torch.fft.fft(x, dim=0)
    w = torch.zeros((nz, 1), dtype=torch.float64, device=DEV)
    w[0] = w[nz // 2] = 1.0
    w[1:nz // 2] = 2.0
    env = torch.fft.ifft(X * w, dim=0).abs()
    db = torch.clamp(20 * torch.log10(torch.clamp(env / env.max(), min=1e-30)), min=-RANGE_DB)
    return env, db


def _exact_metrics(im, dx, t, b, bins):
    im = im.astype(np.float64)
    a, o = im[t[2]:t[3], t[0]:t[1]], im[b[2]:b[3], b[0]:b[1]]
    peak = max(a.max(), o.max())
    h = [np.bincount(np.clip((r.ravel() / peak * bins).astype(int), 0, bins - 1), minlength=bins) / r.size
         for r in (a, o)]
    z, x = np.unravel_index(np.argmax(a), a.shape)
    row, x = im[t[2] + z], t[0] + x
    half, edges = row[x] / 2, []
    for step in (-1, 1):
        j = x
        while 0 <= j + step < row.size and row[j + step] > half:
            j += step
        edges.append(float(j) if not 0 <= j + step < row.size
                     else j + step * (row[j] - half) / (row[j] - row[j + step]))
    mu, mo, so = a.mean(), o.mean(), o.std()
    return {"snr_db": 20 * math.log10(mu / so), "cr_db": 20 * math.log10(mu / mo),
            "gcnr": float(1 - np.minimum(h[0], h[1]).sum()), "fwhm_m": float((edges[1] - edges[0]) * dx),
            "mu_in": float(mu), "mu_out": float(mo), "sigma_out": float(so)}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("frame", "orders"):
        xe, t0, rf, scale = _frame_inputs(case, seed)
        orders = [case["order"]] if kind == "frame" else list(range(1, case["max_order"] + 1))
        out = _exact_frames(case, xe, t0, [rf], [scale], orders, bool(case.get("cf")))[0]
        return out[0] if kind == "frame" else out
    if kind == "batch":
        ins = [_frame_inputs(case, seed, k) for k in range(case["frames"])]
        orders = list(range(case["order_lo"], case["order_hi"] + 1))
        got = _exact_frames(case, ins[0][0], 0.0, [i[2] for i in ins], [i[3] for i in ins], orders)
        return [[got[r][o] for r in range(len(ins))] for o in range(len(orders))]
    if kind in ("mixed", "serve"):
        records, out = {}, []
        for m in _members(case):
            rec = (m["n"], m["s"])
            if rec not in records:
                records[rec] = _frame_inputs(m, seed)
            xe, t0, rf, scale = records[rec]
            out.append(_exact_frames(m, xe, t0, [rf], [scale], [m["order"]])[0][0])
        return out
    if kind == "display":
        got = [_exact_display(im, _taps(case)) for im in _beam_images(case, seed)]
        return ([e for e, _ in got] if case["envelope"] else []) + [d for _, d in got]
    im, target, background = _envelope_image(case, seed)
    return _exact_metrics(im, PITCH / 4, target, background, case["bins"])
