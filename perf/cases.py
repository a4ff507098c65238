"""Workloads whose speed is watched: what programs built on this package do.

Each case is one pass through the public entry points of
``paper_2209_13168_amd.ecmd`` on synthetic ventral-descent events drawn on the
GPU from a seed (the scene of ``synth/ventral.py``: textured surface points
that move radially from the focus of expansion, uniform noise, hot pixels on
the large sensor, coordinate jitter, events sorted by time).  A program keeps
one context, so all cases share it.

Windows of a batch are ragged: their event counts are spaced evenly in the
logarithm between ``n_lo`` and ``n_hi``, in an order drawn from the seed.
Search results are returned with every field of ``ecmd_result``.
"""

from __future__ import annotations

import math
import os
import struct
import tempfile

import numpy as np
import torch

from paper_2209_13168_amd import ecmd, learned

TAU = 0.25
# sensor sizes of the repository's configurations: (width, height, surface
# points, noise share, jitter in pixels, hot-pixel share, largest d searched,
# range of the true d)
SENSORS = {
    "128x128": (128, 128, 300, 0.10, 0.0, 0.0, 1.0, (0.1, 0.8)),
    "346x260": (346, 260, 2000, 0.20, 0.5, 0.0, 1.5, (0.05, 0.8)),
    "640x480": (640, 480, 6830, 0.20, 0.5, 0.0, 1.5, (0.1, 0.6)),
    "1280x720": (1280, 720, 20490, 0.30, 0.5, 0.001, 2.0, (0.05, 1.5)),
}
WEIGHTS = {"1280x720": "cnn_c5.npz"}  # the other sensors use cnn_c2.npz
GRID = 64 * 64


def listed():
    def c(name, kind, sensor="346x260", B=1, n_lo=0, n_hi=0, **kw):
        return dict(name=name, kind=kind, sensor=sensor, B=B, n_lo=n_lo, n_hi=n_hi, **kw)

    return [
        # a control loop: the newest half second of a small sensor, one window
        # per call, where latency and launches count
        c("one_128", "one", "128x128", 1, 10_000, 10_000, eps=1e-4),
        # an ordinary batch of a 346x260 sensor
        c("batch_346", "batch", "346x260", 32, 100_000, 100_000, eps=1e-5),
        # a ragged VGA batch, as a recorded descent gives
        c("batch_640", "batch", "640x480", 64, 50_000, 1_000_000, eps=1e-5),
        # the stress sensor: hot pixels, large windows
        c("batch_1280", "batch", "1280x720", 64, 100_000, 5_000_000, eps=1e-5),
        # proposals of the trained network, Algorithm 1's stop at 0.025
        c("learned_1280", "learned", "1280x720", 12, 100_000, 2_000_000, eps=1e-5, gamma=0.025),
        # a recorded stream in host memory with polarities, cut into windows
        c("stream_pol_346", "stream", "346x260", 10, 60_000, 60_000, eps=1e-5),
        # serving: the asynchronous plan, a few windows a launch
        c("plan_346", "plan", "346x260", 8, 30_000, 120_000, eps=1e-4),
        # a contrast curve of one window: many point hypotheses
        c("curve_346", "curve", "346x260", 1, 100_000, 100_000, m=256),
        # preprocessing: hot pixels removed, then resized and resampled
        c("preproc_1280", "preproc", "1280x720", 16, 200_000, 3_000_000, keep=0.25),
        # proposals for a VGA batch: network input and forward pass
        c("propose_640", "propose", "640x480", 64, 50_000, 1_000_000),
        # gradients of a small training batch
        c("grads_40", "grads", B=40),
        # one training step at the training driver's batch size
        c("train_256", "train", B=256),
    ]


def draw(rng):
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["one", "batch", "batch", "batch", "learned", "stream", "plan", "curve", "preproc", "propose",
                       "grads", "train"])
    if kind in ("grads", "train"):
        return dict(kind=kind, sensor="346x260", B=log(1, 256), n_lo=0, n_hi=0)
    sensor = rng.choice(list(SENSORS))
    top = {"128x128": 30_000, "346x260": 200_000, "640x480": 1_000_000, "1280x720": 3_000_000}[sensor]
    a, b = sorted((log(3_000, top), log(3_000, top)))
    B = log(2, 24 if sensor == "1280x720" else 48)
    eps = rng.choice([1e-4, 1e-5])
    if kind == "one":
        return dict(kind=kind, sensor=sensor, B=1, n_lo=b, n_hi=b, eps=eps)
    if kind == "batch":
        return dict(kind=kind, sensor=sensor, B=B, n_lo=a, n_hi=b, eps=eps)
    if kind == "learned":
        return dict(kind=kind, sensor=sensor, B=min(B, 16), n_lo=a, n_hi=b, eps=eps, gamma=rng.choice([0.0, 0.025]))
    if kind == "stream":
        n = min(b, 150_000)
        return dict(kind=kind, sensor=sensor, B=min(B, 12), n_lo=n, n_hi=n, eps=eps)
    if kind == "plan":
        return dict(kind=kind, sensor=sensor, B=min(B, 8), n_lo=min(a, 200_000), n_hi=min(b, 200_000), eps=eps)
    if kind == "curve":
        return dict(kind=kind, sensor=sensor, B=1, n_lo=min(b, 500_000), n_hi=min(b, 500_000), m=log(4, 400))
    if kind == "preproc":
        return dict(kind=kind, sensor=sensor, B=min(B, 16), n_lo=a, n_hi=b, keep=rng.choice([0.1, 0.25, 0.5]))
    return dict(kind="propose", sensor=sensor, B=B, n_lo=a, n_hi=b)


# ------------------------------------------------------------------ inputs

_shared = {}


def _ctx():
    if "ctx" not in _shared:
        _shared["ctx"] = ecmd.Context(0)
    return _shared["ctx"]


def _weights(sensor):
    path = os.path.join(os.path.dirname(os.path.abspath(learned.__file__)), "weights",
                        WEIGHTS.get(sensor, "cnn_c2.npz"))
    return np.load(path, allow_pickle=False)["params"].astype(np.float32)


def _counts(case):
    """Signal and noise events of every window (hot pixels come on top)."""
    B, lo, hi = case["B"], case["n_lo"], case["n_hi"]
    return [int(round(lo * (hi / lo) ** (k / (B - 1)))) if B > 1 else hi for k in range(B)]


def _hot(case):
    """Hot pixels of the sensor and the events of one in a window (1 kHz)."""
    W, H, hot = SENSORS[case["sensor"]][0], SENSORS[case["sensor"]][1], SENSORS[case["sensor"]][5]
    return int(round(hot * W * H)), int(TAU * 1000)


def _events(case):
    nh, per = _hot(case)
    return sum(_counts(case)) + case["B"] * nh * per


def _below(v, hi):
    return torch.clamp(v.float(), 0.0, float(np.nextafter(np.float32(hi), np.float32(0))))


def _window(case, n, g):
    """x, y, t_rel of one window on the GPU, sorted by time."""
    W, H, points, noise, jitter, _, _, (d0, d1) = SENSORS[case["sensor"]]
    dev = "cuda"

    def uni(k, lo=0.0, hi=1.0):
        return torch.rand(k, generator=g, device=dev, dtype=torch.float64) * (hi - lo) + lo

    cx, cy = W / 2, H / 2
    n_noise = int(round(n * noise))
    ns = n - n_noise
    D = float(uni(1, d0, d1))
    px, py = uni(points, 0, W), uni(points, 0, H)
    w = -torch.log(uni(points) + 1e-12) * (0.25 + torch.hypot(px - cx, py - cy) / math.hypot(cx, cy))
    cum = torch.cumsum(w, 0)
    own = torch.searchsorted(cum, uni(ns) * cum[-1]).clamp_(max=points - 1)
    ts = uni(ns, 0, TAU)
    k = (1 - D * TAU) / (1 - D * ts)
    sx, sy = cx + (px[own] - cx) * k, cy + (py[own] - cy) * k
    if jitter:
        # jitter that would leave the sensor is left out
        jx = sx + jitter * torch.randn(ns, generator=g, device=dev, dtype=torch.float64)
        jy = sy + jitter * torch.randn(ns, generator=g, device=dev, dtype=torch.float64)
        ok = (jx >= 0) & (jx < W) & (jy >= 0) & (jy < H)
        sx, sy = torch.where(ok, jx, sx), torch.where(ok, jy, sy)
    nh, per = _hot(case)
    pix = torch.randperm(W * H, generator=g, device=dev)[:nh]
    th = (uni(nh, 0, TAU / per)[:, None] + torch.arange(per, device=dev)[None] * (TAU / per)).reshape(-1)
    x = torch.cat([sx, uni(n_noise, 0, W), ((pix % W).double() + 0.5).repeat_interleave(per)])
    y = torch.cat([sy, uni(n_noise, 0, H), ((pix // W).double() + 0.5).repeat_interleave(per)])
    t = _below(torch.cat([ts, uni(n_noise, 0, TAU), th]), TAU)
    t, order = torch.sort(t)
    return _below(x[order], W), _below(y[order], H), t


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _batch(case, seed):
    """x, y, t_rel, offsets, tau of the case's windows on the GPU."""
    g = _gen(seed)
    counts = _counts(case)
    order = np.random.default_rng(seed).permutation(len(counts))
    wins = [_window(case, counts[k], g) for k in order]
    off = torch.tensor([0] + [int(w[0].numel()) for w in wins], dtype=torch.int64).cumsum(0).to("cuda")
    x, y, t = (torch.cat([w[i] for w in wins]) for i in range(3))
    return x, y, t, off, torch.full((len(wins),), TAU, dtype=torch.float32, device="cuda")


def _images(B, seed):
    """Network inputs as the downsampling gives them (bfloat16 bits of the
    counts of about 100k events, scaled to mean one) and labels."""
    g = _gen(seed)
    lam = -torch.log(torch.rand(B, GRID, generator=g, device="cuda") + 1e-9) * 0.8 + 0.2
    n = torch.poisson(lam * (100_000 / GRID), generator=g)
    img = (n * (GRID / n.sum(1, keepdim=True))).to(torch.bfloat16)
    return img.view(torch.int16).contiguous(), torch.rand(B, generator=g, device="cuda") * 0.75 + 0.05


def _adam_state(seed):
    """Moments of a training run some way in (v above every m squared)."""
    r = np.random.default_rng(seed)
    v = ((0.5 + r.random(ecmd.CNN_NPARAM)) * 4e-3) ** 2
    m = r.standard_normal(ecmd.CNN_NPARAM) * 1e-3
    return m.astype(np.float32), v.astype(np.float32), 400


LR = 1e-3


def _curve_d(case, seed):
    hi = SENSORS[case["sensor"]][6]
    return np.sort(np.random.default_rng(seed).uniform(0.0, hi, case["m"])).astype(np.float32)


def prepare(case, seed):
    kind = case["kind"]
    ctx = _ctx()
    s = dict(case=case, ctx=ctx)
    if kind in ("grads", "train"):
        s["imgs"], s["labels"] = _images(case["B"], seed)
        s["net"] = ecmd.Cnn(ctx)
        s["net"].set_params(_weights("346x260"))
        if kind == "train":  # a training run taken up again from its checkpoint
            m, v, step = _adam_state(seed)
            with tempfile.TemporaryDirectory() as d:
                path = os.path.join(d, "net.ckpt")
                with open(path, "wb") as f:
                    f.write(b"ECMDCNN1" + struct.pack("<Ii", ecmd.CNN_NPARAM, step))
                    for a in (_weights("346x260"), m, v):
                        f.write(a.tobytes())
                s["net"].load(path)
        return s
    W, H, hi = SENSORS[case["sensor"]][0], SENSORS[case["sensor"]][1], SENSORS[case["sensor"]][6]
    s["sensor"] = ecmd.sensor(W, H, (W / 2, H / 2))
    s["hi"] = hi
    x, y, t, off, tau = _batch(case, seed)
    s.update(x=x, y=y, t=t, off=off, tau=tau)
    if kind == "one":
        s["t"] = t.double() + 100.0
    elif kind == "stream":
        o = off.cpu().numpy()
        k = np.repeat(np.arange(case["B"]), np.diff(o))
        r = np.random.default_rng(seed)
        s["x"], s["y"] = x.cpu().numpy(), y.cpu().numpy()
        s["t"] = 100.0 + TAU * k + t.cpu().numpy().astype(np.float64)
        s["p"] = r.choice(np.array([-1, 1], np.int8), size=o[-1])
    elif kind == "plan":
        s["plan"] = ctx.batch_plan(s["sensor"], 0.0, hi, case["eps"], max_windows=case["B"], max_events=int(x.numel()))
        s["out"] = s["plan"].result_buffer(case["B"])
    elif kind == "curve":
        s["d"] = torch.from_numpy(_curve_d(case, seed)).to("cuda")
    elif kind == "preproc":
        # the resampled events go into the program's own batch buffers
        s["small"] = ecmd.sensor(W // 8, H // 8, (W / 16, H / 16))
        s["seed"] = seed
        s["kept"] = torch.zeros(3, x.numel(), device="cuda")
    if kind in ("learned", "propose"):
        s["net"] = ecmd.Cnn(ctx)
        s["net"].set_params(_weights(case["sensor"]))
    return s


# ---------------------------------------------------------------- one pass

_WHOLE = ("status", "j_star", "L", "n_events", "nodes_expanded", "nodes_pruned", "point_evals", "bound_evals",
          "event_hyp_evals", "pixel_updates", "steps", "seeded", "bound_certs")
_REAL = ("d_hat", "contrast", "d_end", "gap")


def _fields(res):
    out = {f: np.array([getattr(r, f) for r in res], np.int64) for f in _WHOLE}
    out.update({f: np.array([getattr(r, f) for r in res], np.float64) for f in _REAL})
    out["K_hi"] = np.array([r.K >> 62 for r in res], np.int64)
    out["K_lo"] = np.array([r.K & ((1 << 62) - 1) for r in res], np.int64)
    return out


def run(s):
    case, ctx = s["case"], s["ctx"]
    kind = case["kind"]
    if kind == "one":
        return _fields([ctx.estimate(s["sensor"], s["x"], s["y"], s["t"], 100.0, 100.0 + TAU, 0.0, s["hi"],
                                     case["eps"])])
    if kind == "batch":
        return _fields(ctx.estimate_batched(s["sensor"], s["x"], s["y"], s["t"], s["off"], s["tau"], 0.0, s["hi"],
                                            case["eps"]))
    if kind == "learned":
        return _fields(ctx.estimate_learned(s["net"], s["sensor"], s["x"], s["y"], s["t"], s["off"], s["tau"], 0.0,
                                            s["hi"], case["eps"], gamma=case["gamma"]))
    if kind == "stream":
        return _fields(ctx.estimate_stream(s["sensor"], s["x"], s["y"], s["t"], 100.0, TAU, case["B"], 0.0, s["hi"],
                                           case["eps"], polarity=s["p"]))
    if kind == "plan":
        s["plan"].launch(s["x"], s["y"], s["t"], s["off"], s["tau"], s["out"])
        return s["out"]
    if kind == "curve":
        return ctx.probe_point(s["sensor"], s["x"], s["y"], s["t"], TAU, s["d"])
    if kind == "preproc":
        f = ctx.hot_pixel_filter(s["sensor"], s["x"], s["y"], s["t"], s["off"], 50)
        *v, off = ctx.resample(s["sensor"], s["small"], *f, case["keep"], s["seed"])
        for to, a in zip(s["kept"], v):
            to[:a.numel()] = a
        return s["kept"], off
    if kind == "propose":
        imgs = ctx.downsample(s["sensor"], s["x"], s["y"], s["off"])
        return imgs, s["net"].forward(imgs)
    if kind == "grads":
        g, loss = s["net"].grads(s["imgs"], s["labels"])
        return g, np.float32(loss)
    loss = s["net"].train_step(s["imgs"], s["labels"], LR)
    return s["net"].params(), np.float32(loss)


# ----------------------------------------------------- what a pass cannot skip

# Multiplications and additions of one image: forward, and each of the two
# products of the backward pass (the first layer has no input gradient).
_MACS = (16 * 32 * 32 * 9, 32 * 16 * 16 * 16 * 9, 64 * 8 * 8 * 32 * 9)


def work(case):
    kind, B = case["kind"], case["B"]
    if kind in ("grads", "train"):
        macs = 3 * sum(_MACS) - _MACS[0]
        return {"bytes": B * (2 * GRID + 4) + ecmd.CNN_NPARAM * 4 * (6 if kind == "train" else 2),
                "flops": 2.0 * macs * B}
    n = _events(case)
    if kind == "preproc":
        kept = n - B * _hot(case)[0] * _hot(case)[1]
        return {"bytes": 12 * n + 12 * kept * case["keep"], "flops": 2.0 * kept * case["keep"]}
    if kind == "propose":
        return {"bytes": 8 * n + B * 2 * GRID, "flops": 4.0 * n + 2.0 * sum(_MACS) * B}
    if kind == "curve":  # two fused multiply-adds per event and hypothesis
        return {"bytes": 12 * n + 20 * case["m"], "flops": 4.0 * n * case["m"]}
    # Algorithm 1 at least expands the nodes from the root to the optimum: a
    # point and two intervals (two warps each) of every event per level
    L = math.ceil(math.log2(SENSORS[case["sensor"]][6] / case["eps"]))
    per = {"one": 16, "stream": 17}.get(kind, 12)
    return {"bytes": per * n + 160 * B, "flops": 20.0 * n * L}


# ------------------------------------------------------------- 64-bit values


def _bf(v):
    return v + (v.detach().float().to(torch.bfloat16).double() - v.detach())


def _net64(p, imgs):
    """The network in 64 bits: layer inputs and weights rounded to bfloat16."""
    x = imgs.view(torch.bfloat16).double().reshape(-1, 1, 64, 64)
    at = 0
    for co, ci in ((16, 1), (32, 16), (64, 32)):
        w, b = p[at:at + co * ci * 9].reshape(co, ci * 9), p[at + co * ci * 9:at + co * ci * 9 + co]
        at += co * ci * 9 + co
        h = x.shape[-1] // 2
        cols = torch.nn.functional.unfold(_bf(x), 3, padding=1, stride=2)
        x = torch.relu(torch.matmul(_bf(w), cols) + b[:, None]).reshape(-1, co, h, h)
    return _bf(x.mean((2, 3))) @ _bf(p[at:at + 64]) + p[at + 64]


def exact(case, seed):
    """Values in 64 bits.  Searches, curves and the network's input are whole
    numbers by definition (counts of pixels under a stated fp32 warp) and
    their real fields follow from them, so those have no value here."""
    kind = case["kind"]
    if kind in ("grads", "train"):
        imgs, labels = _images(case["B"], seed)
        p = torch.from_numpy(_weights("346x260").astype(np.float64)).to("cuda").requires_grad_()
        loss = ((_net64(p, imgs) - labels.double()) ** 2).mean()
        loss.backward()
        if kind == "grads":
            return p.grad, loss.detach().reshape(())
        m, v, step = _adam_state(seed)
        g = p.grad.cpu().numpy()
        m = 0.9 * m.astype(np.float64) + 0.1 * g
        v = 0.999 * v.astype(np.float64) + 0.001 * g * g
        k = step + 1
        new = p.detach().cpu().numpy() - LR * (m / (1 - 0.9 ** k)) / (np.sqrt(v / (1 - 0.999 ** k)) + 1e-8)
        return new, loss.detach().reshape(())
    if kind == "propose":
        x, y, _, off, _ = _batch(case, seed)
        W, H = SENSORS[case["sensor"]][:2]
        win = torch.repeat_interleave(torch.arange(case["B"], device="cuda"), off[1:] - off[:-1])
        bx = torch.floor(x * 64.0 / W).long().clamp(0, 63)
        by = torch.floor(y * 64.0 / H).long().clamp(0, 63)
        cnt = torch.bincount(win * GRID + by * 64 + bx, minlength=case["B"] * GRID).reshape(-1, GRID)
        img = (cnt.float() * (4096.0 / (off[1:] - off[:-1]).float())[:, None]).to(torch.bfloat16)
        p = torch.from_numpy(_weights(case["sensor"]).astype(np.float64)).to("cuda")
        return None, _net64(p, img)
    if kind == "preproc":
        x, y, t, off, _ = _batch(case, seed)
        W, H = SENSORS[case["sensor"]][:2]
        B = case["B"]
        win = torch.repeat_interleave(torch.arange(B, device="cuda"), off[1:] - off[:-1])
        pix = win * (W * H) + y.long() * W + x.long()
        keep = torch.bincount(pix, minlength=B * W * H)[pix] <= 50
        f = (x[keep], y[keep], t[keep])
        n = torch.bincount(win[keep], minlength=B)
        first = torch.cumsum(n, 0) - n
        w = win[keep]
        ctr = (w << 32) + (torch.arange(w.numel(), device="cuda") - first[w]) + 1
        z = ctr.cpu().numpy().astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15) + np.uint64(seed)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = (z ^ (z >> np.uint64(31))) >> np.uint64(40)
        k = torch.from_numpy(z < np.uint64(math.floor(np.float32(case["keep"]) * 16777216.0))).to("cuda")
        out = torch.zeros(3, x.numel(), dtype=torch.float64, device="cuda")
        for to, v, scale in zip(out, f, ((W // 8) / W, (H // 8) / H, 1.0)):
            to[:int(k.sum())] = v[k].double() * scale
        return out, None
    return None
