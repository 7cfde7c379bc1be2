"""Performance cases of the framework, each through the entry points that a program calls.

A case is a dict of plain values. `listed()` gives the fixed ones, `draw(rng)` one more of the same ranges,
`prepare(case, seed)` what a program holds before the call (resident scenes, positions, targets), `run(state)` one
pass and its outputs, `work(case)` the bytes and operations that a pass cannot do without, and `exact(case, seed)`
the same outputs in 64 bits from plain torch.

Kinds of work:
  render   spectra of one resident scene for a batch of transmitter positions (BF16 or FP32 deformation MLP, or the
           static scene), optionally with a periodic azimuth or on another resolution of the same field of view
  mixed    one launch sequence over queries of several resident scenes (what the serving loop launches)
  rssi     the RSSI head: one pooled value per position from a small spectrum
  paper    the paper's own model (order-free sum, 8 x 156 MLP), magnitude and both channels
  train    forward with the blend state kept, hybrid loss, backward to every parameter (autograd)
  beamscan target spectra from multipath lists
"""
import math
import time

import numpy as np
import torch

from paper_2506_12787_amd import binding as B
from paper_2506_12787_amd import synth
from paper_2506_12787_amd.autograd import Renderer

ROOM = ((0.0, 0.0, 0.0), (6.0, 6.0, 3.0))
FLAGS = {"bf16": B.MLP_BF16, "fp32": B.MLP_FP32, "static": B.NO_DEFORM}
MLP_FLOPS = 2 * (26 * 256 + 3 * 256 * 256 + 256 * 7)  # per (position, Gaussian) pair, layer 1's position part once
MLP_BWD_FLOPS = 2 * MLP_FLOPS  # input and weight gradients of every layer
PAPER_FLOPS = 2 * (81 * 156 + 4 * 156 * 156 + 3 * 237 * 156 + 156 * 5)
MLP_BYTES = 4 * (89 * 256 + 3 * 256 * 256 + 256 * 7 + 4 * 256 + 7)
EXACT_SECONDS = 18.0


def listed():
    return [
        # one position of an online RSSI localiser (the smallest call: latency and launches)
        {"name": "rssi_one", "kind": "rssi", "mlp": "bf16", "n": 50, "h": 16, "w": 16, "batch": 1},
        # the RSSI head over a fingerprint grid: many queries of very few Gaussians each
        {"name": "rssi_batch", "kind": "rssi", "mlp": "bf16", "n": 50, "h": 16, "w": 16, "batch": 1024},
        # an interactive query at full precision: one position, one launch sequence
        {"name": "query_fp32", "kind": "render", "mlp": "fp32", "n": 100_000, "h": 90, "w": 360, "batch": 1},
        # a few waiting requests of a mid-sized scene; odd sizes, tiles cut by the grid's edge, seam at 0/360 degrees
        {"name": "few_ragged", "kind": "render", "mlp": "bf16", "n": 20_011, "h": 91, "w": 361, "batch": 5,
         "wrap": True},
        # saturated serving of one scene (the benchmark's default workload)
        {"name": "batch_dense", "kind": "render", "mlp": "bf16", "n": 100_000, "h": 90, "w": 360, "batch": 64},
        # half-degree maps of a one-degree scene
        {"name": "map_hires", "kind": "render", "mlp": "bf16", "n": 50_000, "h": 90, "w": 360, "batch": 16, "scale": 2},
        # the large scene of the benchmark, a quarter of its batch
        {"name": "scene_large", "kind": "render", "mlp": "bf16", "n": 500_000, "h": 360, "w": 1440, "batch": 64,
         "lo": 0.5, "hi": 20.0},
        # a serving launch over several resident scenes of different sizes
        {"name": "mixed_scenes", "kind": "mixed", "mlp": "bf16", "batch": 64, "scenes": 4, "n": 100_000},
        # the paper's model at the paper's size
        {"name": "paper_model", "kind": "paper", "n": 10_000, "h": 90, "w": 360, "batch": 64},
        # training: the benchmark's BF16 step, and full precision at the paper's Gaussian count
        {"name": "train_bf16", "kind": "train", "mlp": "bf16", "n": 50_000, "h": 90, "w": 360, "batch": 16},
        {"name": "train_fp32", "kind": "train", "mlp": "fp32", "n": 10_000, "h": 90, "w": 360, "batch": 16},
        # target spectra for a training set
        {"name": "beam_targets", "kind": "beamscan", "side": 4, "h": 90, "w": 360, "batch": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["render", "render", "render", "mixed", "rssi", "paper", "train", "train", "beamscan"])
    c = {"kind": kind}
    if kind == "rssi":
        side = rng.choice([12, 16, 24, 32])
        c.update(mlp=rng.choice(["bf16", "fp32"]), n=_log_int(rng, 20, 400), h=side, w=side,
                 batch=_log_int(rng, 1, 2048))
        return c
    if kind == "mixed":
        c.update(mlp=rng.choice(["bf16", "bf16", "static", "fp32"]), batch=rng.randint(2, 64),
                 scenes=rng.randint(2, 6))
        c["n"] = _log_int(rng, 5_000, 20_000 if c["mlp"] == "fp32" else 150_000)
        return c
    if kind == "beamscan":
        c.update(side=rng.choice([2, 3, 4, 5, 6, 8]), batch=_log_int(rng, 1, 512))
        c["h"], c["w"] = rng.choice([(90, 360), (91, 361), (45, 180), (30, 121)])
        return c
    c["h"], c["w"] = rng.choice([(90, 360), (90, 360), (91, 361), (60, 240), (45, 181), (100, 400)])
    if kind == "paper":
        c.update(n=_log_int(rng, 1_000, 20_000), batch=_log_int(rng, 1, 64))
        return c
    if kind == "train":
        c.update(mlp=rng.choice(["bf16", "fp32"]), n=_log_int(rng, 2_000, 50_000), batch=_log_int(rng, 1, 16))
        if rng.random() < 0.25:
            c["deterministic"] = True
        if rng.random() < 0.25:
            c["wrap"] = True
        return c
    c["mlp"] = rng.choice(["bf16", "bf16", "bf16", "fp32", "static"])
    c["n"] = _log_int(rng, 1_000, 200_000)
    c["batch"] = min(_log_int(rng, 1, 64), max(1, (1_000_000 if c["mlp"] == "fp32" else 6_400_000) // c["n"]))
    more = rng.random()
    if more < 0.25:
        c["wrap"] = True
    elif more < 0.5:
        c["scale"] = 2
    return c


# ---- what a program holds before the call -----------------------------------
_context = None


def _lib():
    """The program's one context on the GPU (a program keeps it for its lifetime)."""
    global _context
    if _context is None:
        _context = B.Context(0)
    return _context


class _Scene:
    """A resident scene, released with the state that holds it."""

    def __init__(self, sid):
        self.sid = sid

    def __del__(self):
        if _context is not None and getattr(_context, "_h", None):
            _context.release_scene(self.sid)


def _scene_inputs(c, seed, n, h, w):
    lo, hi = (0.7, 4.0) if c["kind"] == "rssi" else (c.get("lo", 1.0), c.get("hi", 12.0))
    return synth.gaussians(n, h, w, seed=seed, scale_range=(lo, hi)), synth.mlp_weights(seed=seed + 1)


def _positions(c, seed):
    return synth.tx_positions(c["batch"], seed=seed + 2, room=ROOM)


def _mixed_plan(c):
    """(n, h, w) of every resident scene and the scene of every query."""
    n = c["n"]
    kinds = [(n, 90, 360), (max(n // 5, 1), 180, 720), (max(n // 20, 1), 90, 360), (max(n // 5, 1), 90, 360),
             (max(n // 3, 1), 91, 361), (max(n // 20, 1), 180, 720)]
    r = np.random.default_rng(c["n"])
    return kinds[:c["scenes"]], [int(x) for x in r.integers(0, c["scenes"], c["batch"])]


def _targets(c, seed):
    """Smooth spectra in [0, 1]: a few lobes each, as measured and synthesised ones are."""
    r = np.random.default_rng(seed + 4)
    y, x = np.arange(c["h"])[:, None], np.arange(c["w"])[None, :]
    out = np.zeros((c["batch"], c["h"], c["w"]))
    for b in range(c["batch"]):
        for _ in range(8):
            cy, cx, s = r.uniform(0, c["h"]), r.uniform(0, c["w"]), r.uniform(3, 30)
            out[b] += r.uniform(0.1, 0.5) * np.exp(-((y - cy) ** 2 + (x - cx) ** 2) / (2 * s * s))
    return np.minimum(out, 1.0).astype(np.float32)


def prepare(c, seed):
    lib, kind = _lib(), c["kind"]
    s = {"case": c, "lib": lib}
    if kind == "beamscan":
        paths, counts, _ = synth.multipath(c["batch"], seed=seed)
        s["paths"], s["counts"] = torch.from_numpy(paths).cuda(), torch.from_numpy(counts).cuda()
        return s
    s["tx"] = torch.from_numpy(_positions(c, seed)).cuda()
    if kind == "paper":
        s["scene"] = _Scene(lib.upload_paper_scene(synth.paper_gaussians(c["n"], seed=seed), c["h"], c["w"],
                                                   mlp=synth.paper_mlp_weights(seed=seed + 1, out_scale=0.3),
                                                   room=ROOM))
        return s
    if kind == "mixed":
        kinds, which = _mixed_plan(c)
        s["scenes"] = []
        for i, (n, h, w) in enumerate(kinds):
            g, mlp = _scene_inputs(c, seed + 100 * (i + 1), n, h, w)
            s["scenes"].append(_Scene(lib.upload_scene(g, h, w, mlp=mlp, room=ROOM)))
        s["ids"] = [s["scenes"][i].sid for i in which]
        s["flags"] = FLAGS[c["mlp"]]
        return s
    g, mlp = _scene_inputs(c, seed, c["n"], c["h"], c["w"])
    s["flags"] = FLAGS[c["mlp"]] | (B.WRAP_AZIMUTH if c.get("wrap") else 0)
    if kind == "train":
        s["flags"] |= B.DETERMINISTIC if c.get("deterministic") else 0
        s["model"] = Renderer(g, c["h"], c["w"], mlp=mlp, lib=lib, room=ROOM)
        s["scene"] = _Scene(s["model"].sid)
        s["target"] = torch.from_numpy(_targets(c, seed)).cuda()
        return s
    s["scene"] = _Scene(lib.upload_scene(g, c["h"], c["w"], mlp=mlp if c["mlp"] != "static" else None, room=ROOM))
    return s


def run(s):
    c, lib = s["case"], s["lib"]
    kind = c["kind"]
    if kind == "beamscan":
        return lib.beamscan(s["paths"], s["counts"], c["h"], c["w"], side=c["side"])
    if kind == "paper":
        return lib.render_paper(s["scene"].sid, s["tx"])
    if kind == "mixed":
        return lib.render_mixed(s["ids"], s["tx"] if c["mlp"] != "static" else None, flags=s["flags"])
    if kind == "rssi":
        return lib.render_rssi(s["scene"].sid, s["tx"], flags=s["flags"])
    if kind == "train":
        m = s["model"]
        out = m(s["tx"], flags=s["flags"])
        loss, g = lib.hybrid_loss(out.detach(), s["target"])
        grads = torch.autograd.grad(out, list(m.parameters()), g)
        return {"spectra": out.detach(), "loss": loss, "grads": list(grads)}
    tx, batch = (s["tx"], None) if c["mlp"] != "static" else (None, c["batch"])
    if c.get("scale"):
        return lib.render_at(s["scene"].sid, c["h"] * c["scale"], c["w"] * c["scale"], tx, flags=s["flags"],
                             batch=batch)
    return lib.render(s["scene"].sid, tx, flags=s["flags"], batch=batch)


# ---- the least a pass needs --------------------------------------------------
def work(c):
    kind, nb = c["kind"], c["batch"]
    if kind == "beamscan":
        return {"bytes": 4.0 * nb * (75 + c["h"] * c["w"]), "flops": 8.0 * c["side"] ** 2 * nb * c["h"] * c["w"]}
    if kind == "mixed":
        kinds, which = _mixed_plan(c)
        pairs = sum(kinds[i][0] for i in which)
        values = sum(kinds[i][1] * kinds[i][2] for i in which)
        scenes = sum(n for n, _, _ in kinds)
        per = 0 if c["mlp"] == "static" else MLP_FLOPS
        return {"bytes": 4.0 * (7 * scenes + values) + (MLP_BYTES * len(kinds) if per else 0),
                "flops": float(pairs) * (per + 100)}
    pairs, values = float(nb) * c["n"], float(nb) * c["h"] * c["w"] * c.get("scale", 1) ** 2
    if kind == "paper":
        return {"bytes": 32.0 * c["n"] + 4.0 * 222_929 + 12.0 * values, "flops": pairs * (PAPER_FLOPS + 100)}
    if kind == "rssi":
        return {"bytes": 28.0 * c["n"] + MLP_BYTES + 16.0 * nb, "flops": pairs * (MLP_FLOPS + 100)}
    if kind == "train":
        # parameters in and gradients out, targets in, spectra out
        return {"bytes": 2.0 * (28 * c["n"] + MLP_BYTES) + 8.0 * values,
                "flops": pairs * (MLP_FLOPS + MLP_BWD_FLOPS + 200)}
    per = 0 if c["mlp"] == "static" else MLP_FLOPS
    return {"bytes": 28.0 * c["n"] + (MLP_BYTES if per else 0) + 12.0 * nb + 4.0 * values,
            "flops": pairs * (per + 100)}


# ---- the same outputs in 64 bits ----------------------------------------------
def _d(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.float64, device="cuda")


def _features(v, bands):
    """[v, sin(2^k pi v), cos(2^k pi v)] over the components of v (rows, components)."""
    f = [v] + [torch.sin(2.0 ** k * math.pi * v) for k in range(bands)]
    return torch.cat(f + [torch.cos(2.0 ** k * math.pi * v) for k in range(bands)], 1)


def _unit_tx(tx):
    lo, hi = _d(ROOM[0]), _d(ROOM[1])
    return (_d(tx) - lo) / (hi - lo)


def _residuals(mu, tx, Ws, bs):
    """Residuals (n, 7) of one position; mu (n, 2) in units of the grid."""
    fs = _features(tx[None, :], 10).expand(mu.shape[0], -1)
    x = torch.cat([_features(mu, 6), fs], 1)
    for w, b in zip(Ws[:-1], bs[:-1]):
        x = torch.relu(x @ w.T + b)
    return x @ Ws[-1].T + bs[-1]


A_MAX, A_MIN, T_MIN = float(np.float32(0.99)), float(np.float32(1.0) / np.float32(255.0)), float(np.float32(1e-4))


def _chunk_alpha(p, xs, ys, period):
    """alpha (Gaussians, pixels) of deformed parameters p (g, 7) with the cutoff, clamp and skip applied."""
    mx, my, lsx, lsy, rot, logit = (p[:, k:k + 1] for k in range(6))
    dx, dy = xs - mx, ys - my
    if period:
        dx = dx - period * torch.round(dx.detach() / period)
    co, si = torch.cos(rot), torch.sin(rot)
    u, v = (co * dx + si * dy) * torch.exp(-lsx), (co * dy - si * dx) * torch.exp(-lsy)
    q = u * u + v * v
    a = torch.clamp(torch.sigmoid(logit) * torch.exp(-0.5 * q), max=A_MAX)
    return torch.where((q <= 9.0) & (a >= A_MIN), a, torch.zeros_like(a))


class _TooLong(Exception):
    pass


def _composite(p, h, w, sx, sy, period, until, grad=None):
    """Spectrum (h * w) of parameters p (n, 7 + amplitude last) in depth order; with `grad` (h * w) the gradient of
    sum(grad * spectrum) with respect to p instead, every decision held."""
    ys, xs = torch.meshgrid(torch.arange(h, device="cuda", dtype=torch.float64) / sy,
                            torch.arange(w, device="cuda", dtype=torch.float64) / sx, indexing="ij")
    xs, ys = xs.reshape(1, -1), ys.reshape(1, -1)
    size = max(64, (1 << 25) // (h * w))
    spectrum = _composite(p, h, w, sx, sy, period, until) if grad is not None else None
    T, C = torch.ones(h * w, dtype=torch.float64, device="cuda"), torch.zeros(h * w, dtype=torch.float64, device="cuda")
    dp = torch.zeros_like(p) if grad is not None else None
    for at in range(0, p.shape[0], size):
        if time.time() > until:
            raise _TooLong()
        pc = p[at:at + size].detach()
        with torch.set_grad_enabled(grad is not None):
            pc.requires_grad_(grad is not None)
            a = _chunk_alpha(pc, xs, ys, period)
        al = a.detach()
        Tn = T * torch.cumprod(1.0 - al, 0)
        Tp = torch.cat([T[None], Tn[:-1]])
        live = Tn >= T_MIN
        amp = pc.detach()[:, 6:7]
        add = torch.where(live, amp * al * Tp, torch.zeros_like(al))
        if grad is not None:
            after = spectrum - (C + torch.cumsum(add, 0))  # what the entries behind add
            ga = torch.where(live & (al > 0), grad * (amp * Tp - after / (1.0 - al)), torch.zeros_like(al))
            dp[at:at + size] = torch.autograd.grad(a, pc, ga)[0]
            dp[at:at + size, 6] = (torch.where(live, al * Tp, torch.zeros_like(al)) * grad).sum(1)
        C, T = C + add.sum(0), Tn[-1]
        if float(T.max()) < T_MIN:
            break
    return dp if grad is not None else C


def _exact_scene(c, g, mlp, tx, h, w, scale, until, grads_of=None):
    """Spectra (len(tx), h * scale, w * scale); with `grads_of(spectra)` also the gradients it asks for."""
    order = np.argsort(g["depth"], kind="stable")
    keys = synth.PARAM_NAMES[:7]
    base = torch.stack([_d(g[k][order]) for k in keys], 1)
    Ws, bs = [_d(x) for x in mlp[0]], [_d(x) for x in mlp[1]]
    H, W = h * scale, w * scale
    period = float(W) / scale if c.get("wrap") else 0.0
    size = _d([w, h])
    unit = _unit_tx(tx)

    def deformed(i, b, ws, bb):
        if c["mlp"] == "static":
            return b
        return b + _residuals(b[:, :2] / size, unit[i], ws, bb)

    spectra = []
    with torch.no_grad():
        for i in range(len(tx)):
            spectra.append(_composite(deformed(i, base, Ws, bs), H, W, scale, scale, period, until).reshape(H, W))
            if c["mlp"] == "static":
                spectra = spectra * len(tx)
                break
    spectra = torch.stack(spectra)
    if grads_of is None:
        return spectra
    loss, gout = grads_of(spectra)
    leaves = [base.clone().requires_grad_()] + [x.clone().requires_grad_() for x in Ws + bs]
    total = [torch.zeros_like(x) for x in leaves]
    for i in range(len(tx)):
        p = deformed(i, leaves[0], leaves[1:1 + len(Ws)], leaves[1 + len(Ws):])
        dp = _composite(p.detach(), H, W, scale, scale, period, until, gout[i].reshape(-1))
        for t, x in zip(total, torch.autograd.grad(p, leaves, dp)):
            t += x
    inv = torch.from_numpy(np.argsort(order)).cuda()
    return spectra, loss, [total[0][inv, k] for k in range(7)] + total[1:]


def _hybrid(target):
    """(loss (3,), gradient) of 0.7 l1 + 0.3 (1 - SSIM) against `target`."""
    t = _d(target)
    win = torch.exp(-torch.arange(-5, 6, device="cuda", dtype=torch.float64) ** 2 / (2 * 1.5 * 1.5))
    win = win / win.sum()

    def blur(v):
        v = torch.nn.functional.pad(v, (5, 5, 5, 5))
        v = sum(win[k] * v[:, :, k:k + v.shape[2] - 10] for k in range(11))
        return sum(win[k] * v[:, k:k + v.shape[1] - 10] for k in range(11))

    def of(spectra):
        x = spectra.detach().requires_grad_()
        mx, my = blur(x), blur(t)
        vx, vy, cxy = blur(x * x) - mx * mx, blur(t * t) - my * my, blur(x * t) - mx * my
        ssim = ((2 * mx * my + 1e-4) * (2 * cxy + 9e-4) / ((mx * mx + my * my + 1e-4) * (vx + vy + 9e-4))).mean()
        l1 = (x - t).abs().mean()
        loss = 0.7 * l1 + 0.3 * (1 - ssim)
        g, = torch.autograd.grad(loss, x)
        return torch.stack([loss, l1, ssim]).detach(), g

    return of


def _exact_paper(c, seed, until):
    g = synth.paper_gaussians(c["n"], seed=seed)
    Ws, bs = synth.paper_mlp_weights(seed=seed + 1, out_scale=0.3)
    Ws, bs = [_d(x) for x in Ws], [_d(x) for x in bs]
    unit, h, w = _unit_tx(_positions(c, seed)), c["h"], c["w"]
    v = {k: _d(g[k]) for k in synth.PAPER_KEYS}
    mu = torch.stack([0.5 * w * (torch.tanh(v["center_x"]) + 1), 0.5 * h * (torch.tanh(v["center_y"]) + 1)], 1)
    fm = _features(mu / _d([w, h]), 10)
    xs = torch.arange(w, device="cuda", dtype=torch.float64).repeat(h)[None]
    ys = torch.arange(h, device="cuda", dtype=torch.float64).repeat_interleave(w)[None]
    size = max(64, (1 << 25) // (h * w))
    out = torch.zeros((c["batch"], 2, h * w), dtype=torch.float64, device="cuda")
    for i in range(c["batch"]):
        x = torch.cat([fm, _features(unit[i][None], 6).expand(c["n"], -1)], 1)
        a = x
        for l in range(8):
            a = torch.relu((torch.cat([a, x], 1) if l in (2, 4, 6) else a) @ Ws[l].T + bs[l])
        d = a @ Ws[8].T + bs[8]
        gate = torch.sigmoid(v["atten_logit"]) + d[:, 4]
        wre, wim = (v["psi_re"] + d[:, 2]) * gate, (v["psi_im"] + d[:, 3]) * gate
        for at in range(0, c["n"], size):
            if time.time() > until:
                raise _TooLong()
            s = slice(at, at + size)
            dx, dy = xs - (mu[s, 0] + d[s, 0])[:, None], ys - (mu[s, 1] + d[s, 1])[:, None]
            u = dx / v["chol_l1"][s, None]
            t = (dy - v["chol_l2"][s, None] * u) / v["chol_l3"][s, None]
            q = u * u + t * t
            k = torch.where(q <= 9.0, torch.exp(-0.5 * q), torch.zeros_like(q))
            out[i, 0] += wre[s] @ k
            out[i, 1] += wim[s] @ k
    out = out.reshape(c["batch"], 2, h, w)
    return torch.hypot(out[:, 0], out[:, 1]), out


def _exact_beamscan(c, seed):
    paths, counts, _ = synth.multipath(c["batch"], seed=seed)
    p, K = _d(paths), c["side"]
    m = torch.arange(K, device="cuda", dtype=torch.float64)

    def phase(theta, phi):  # element (m, n), m-major, half a wavelength apart
        a = (m[None, :] * torch.cos(theta)[:, None])[:, None, :] + (m[None, :] * torch.sin(theta)[:, None])[:, :, None]
        return -math.pi * (torch.cos(phi)[:, None, None] * a).reshape(-1, K * K)

    y = torch.arange(c["h"], device="cuda", dtype=torch.float64).repeat_interleave(c["w"]) / c["h"]
    x = torch.arange(c["w"], device="cuda", dtype=torch.float64).repeat(c["h"]) / c["w"]
    steer = torch.exp(-1j * phase(2 * math.pi * x, 0.5 * math.pi * y))
    out = []
    for b in range(c["batch"]):
        q = p[b, :int(counts[b])]
        ch = (q[:, :1] * torch.exp(1j * phase(q[:, 1], q[:, 2]))).sum(0)
        out.append((steer @ (ch / ch.abs())).abs() / (K * K))
    return torch.stack(out).reshape(c["batch"], c["h"], c["w"])


def exact(c, seed):
    kind, until = c["kind"], time.time() + EXACT_SECONDS
    try:
        if kind == "beamscan":
            return _exact_beamscan(c, seed)
        if kind == "paper":
            return _exact_paper(c, seed, until)
        tx = _positions(c, seed)
        if kind == "mixed":
            kinds, which = _mixed_plan(c)
            made, out = {}, []
            for i, k in enumerate(which):
                n, h, w = kinds[k]
                if k not in made:
                    made[k] = _scene_inputs(c, seed + 100 * (k + 1), n, h, w)
                out.append(_exact_scene(c, *made[k], tx[i:i + 1], h, w, 1, until)[0])
            return out
        if c["n"] * c["batch"] * c["h"] * c["w"] > 1 << 42:
            return None
        g, mlp = _scene_inputs(c, seed, c["n"], c["h"], c["w"])
        if kind == "train":
            spectra, loss, grads = _exact_scene(c, g, mlp, tx, c["h"], c["w"], 1, until, _hybrid(_targets(c, seed)))
            # a BF16 network's own weight gradient is not that of the 64-bit network
            grads = grads[:7] + ([None] * len(grads[7:]) if c["mlp"] == "bf16" else grads[7:])
            return {"spectra": spectra, "loss": loss, "grads": grads}
        out = _exact_scene(c, g, mlp, tx, c["h"], c["w"], c.get("scale", 1), until)
        return out.mean((1, 2)) if kind == "rssi" else out
    except _TooLong:
        return None
