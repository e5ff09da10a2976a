"""The work a program gives this framework, as a set of timed cases.

Five kinds of call, each through the public entry points of
`paper_2308_09209_amd`:

* ``stitch``  one panorama per pass from one rig (``Stitcher.stitch``): plain
  Lucas-Kanade flow, learned surrogate with fallback, or variational flow;
* ``batch``   one step of several uneven streams (``Batch.run``);
* ``flow``    the plain or variational flow of one luma pair, both directions
  (``PlainFlow``: training labels, or flow without stitching);
* ``train``   one training step of the surrogate (``surrogate.Net``);
* ``conv``    one 3x3 convolution of the network (``vs_nn_conv3x3``).

Sizes are those of the scenes, the benchmark and the training script of this
repository; ``draw`` spreads over the ranges they span.
"""
import ctypes as C
import math
import os
import struct

import torch
import torch.nn.functional as F

from paper_2308_09209_amd import surrogate as S
from paper_2308_09209_amd import vstitch as V

WEIGHTS = os.path.join(os.path.dirname(os.path.abspath(V.__file__)), "weights", "flow_surrogate.vsnn")
FB_TAU = 0.5        # the benchmark's forward-backward threshold (px)
LR = 2e-3           # the training script's learning rate
LEVELS, ITERS, RADIUS, LAMBDA = 4, 5, 4, 256.0   # vs_default_params' flow
DEV = "cuda"


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the smallest rig, one frame at a time, the colour state read back after each (a program
        # that checkpoints its state, or one stream at low latency): launches and waits count
        dict(name="stitch_2x640x360_state", kind="stitch", cams=2, w=640, h=360, overlap=0.30, ring=False,
             flow="plain", state=True),
        # the headline workload: a 360-degree ring of four 1080p cameras
        dict(name="stitch_4x1080p_ring", kind="stitch", cams=4, w=1920, h=1080, overlap=0.20, ring=True,
             flow="plain", state=False),
        # the same with the learned surrogate and its forward-backward fallback
        dict(name="stitch_4x1080p_ring_surrogate", kind="stitch", cams=4, w=1920, h=1080, overlap=0.20, ring=True,
             flow="surrogate", state=False),
        # the same with the variational flow
        dict(name="stitch_4x1080p_ring_var", kind="stitch", cams=4, w=1920, h=1080, overlap=0.20, ring=True,
             flow="variational", state=False),
        # an odd chain of three cameras, surrogate
        dict(name="stitch_3x1277x719_surrogate", kind="stitch", cams=3, w=1277, h=719, overlap=0.25, ring=False,
             flow="surrogate", state=False),
        # the largest rig: eight 4K cameras
        dict(name="stitch_8x4k_ring", kind="stitch", cams=8, w=3840, h=2160, overlap=0.20, ring=True,
             flow="plain", state=False),
        dict(name="stitch_8x4k_ring_surrogate", kind="stitch", cams=8, w=3840, h=2160, overlap=0.20, ring=True,
             flow="surrogate", state=False),
        # six uneven streams (2 x 720p, 2 x 1080p, 2 x 1440p, 3 and 4 cameras), one captured graph per step
        dict(name="batch_6_streams", kind="batch", streams=6, w=1280, step=640, flow="plain"),
        # one training pair's labels (a strip pair of the 1080p ring)
        dict(name="flow_256x1080", kind="flow", w=256, h=1080, flow="plain"),
        # a small odd pair: every level smaller than a tile
        dict(name="flow_97x61", kind="flow", w=97, h=61, flow="plain"),
        # one training step: 16 pairs at level 2 of 256 x 1080
        dict(name="train_16x64x270", kind="train", n=16, w=64, h=270),
        # one 32 -> 32 layer on level-0 strips
        dict(name="conv_32_32_8x256x1080", kind="conv", n=8, w=256, h=1080, cin=32, cout=32, mode="lrelu"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["stitch", "stitch", "stitch", "stitch", "batch", "flow", "flow", "train", "conv"])
    if kind == "stitch":
        flow = rng.choice(["plain", "plain", "surrogate", "variational"])
        cams = rng.randint(2, 8) if flow != "variational" else rng.randint(2, 4)
        w = _log(rng, 320, 3840 if flow != "variational" else 1920)
        h = max(200, int(w * rng.uniform(0.45, 0.5625)))
        ring = cams >= 3 and rng.random() < 0.5
        return dict(kind="stitch", cams=cams, w=w, h=h, overlap=round(rng.uniform(0.2, 0.3), 3), ring=ring, flow=flow,
                    state=rng.random() < 0.25)
    if kind == "batch":
        w = _log(rng, 480, 1280)
        return dict(kind="batch", streams=rng.randint(2, 6), w=w, step=rng.randint(0, w // 2),
                    flow=rng.choice(["plain", "surrogate"]))
    if kind == "flow":
        return dict(kind="flow", w=_log(rng, 48, 520), h=_log(rng, 48, 2160), flow=rng.choice(["plain", "plain", "variational"]))
    if kind == "train":
        return dict(kind="train", n=rng.randint(1, 32), w=_log(rng, 24, 96), h=_log(rng, 60, 400))
    cin, cout = rng.choice([(16, 32), (32, 32), (32, 16)])
    return dict(kind="conv", n=rng.randint(1, 8), w=_log(rng, 32, 300), h=_log(rng, 64, 1200), cin=cin, cout=cout,
                mode=rng.choice(["lrelu", "linear", "f32"]))


# ---------------------------------------------------------------------------
# Inputs: rigs, frames and luma pairs of the scene recipe, made on the device
# ---------------------------------------------------------------------------

def _u(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, dtype=torch.float64)


class _Texture:
    """0.5 + 16 sinusoids per channel, then flat rectangles; periodic in x for a ring."""

    def __init__(self, g, width, height, period, channels, rects=40):
        theta, lam = _u(g, 0.0, math.pi, 16), torch.exp(_u(g, math.log(8.0), math.log(128.0), 16))
        kx, ky = 2 * math.pi * torch.cos(theta) / lam, 2 * math.pi * torch.sin(theta) / lam
        if period:
            kx = torch.round(kx * period / (2 * math.pi)) * (2 * math.pi / period)
        self.kx, self.ky, self.ph = kx.tolist(), ky.tolist(), _u(g, 0.0, 2 * math.pi, 16).tolist()
        self.amp = _u(g, 0.0, 1.0 / 16.0, 16, channels).float().to(DEV)
        self.period = period
        self.reach = 3.0 * math.sqrt(float((self.amp ** 2).sum(0).max()) / 2) + 1e-3
        box = _u(g, 0.0, 1.0, rects, 4)
        self.rects = [(float(a) * width, float(b) * height, 16 + float(c) * max(1.0, height / 4 - 16),
                       16 + float(d) * max(1.0, height / 4 - 16)) for a, b, c, d in box]
        self.cols = _u(g, 0.0, 1.0, rects, channels).float().to(DEV)

    def __call__(self, X, Y):
        v = torch.zeros(X.shape + (self.amp.shape[1],), dtype=torch.float32, device=DEV)
        for i in range(16):
            v += torch.sin((self.kx[i] * X + self.ky[i] * Y + self.ph[i]).float())[..., None] * self.amp[i]
        v = (v / (2 * self.reach) + 0.5).clamp_(0, 1)
        for (x0, y0, rw, rh), col in zip(self.rects, self.cols):
            dx = X - x0
            if self.period:
                dx = torch.remainder(dx, float(self.period))
            inside = (dx >= 0) & (dx < rw) & (Y >= y0) & (Y < y0 + rh)
            v = torch.where(inside[..., None], col, v)
        return v


def _smooth(g, w, h, cell, reach):
    """a smooth random displacement (2, h, w), at most `reach` px long"""
    coarse = torch.randn(1, 2, max(2, h // cell), max(2, w // cell), generator=g).to(DEV)
    d = F.interpolate(coarse, size=(h, w), mode="bicubic", align_corners=True)[0]
    return d * (reach / d.norm(dim=0).max().clamp_min(1e-6))


def _rig(case, stream=0):
    """The installation: cameras at the nominal spacing, each a little rotated, scaled, shifted and tilted."""
    n, w, h = case["cams"], case["w"], case["h"]
    g = torch.Generator().manual_seed(1000 + 10 * stream + n)
    step = int(round(w * (1.0 - case["overlap"])))
    tilt = 1e-4 * min(1.0, 1920.0 / w)
    cx, cy = (w - 1) / 2.0, (h - 1) / 2.0
    Hs = []
    for k in range(n):
        th, s = math.radians(float(_u(g, -3, 3, 1))), float(_u(g, 0.98, 1.02, 1))
        t, p = _u(g, -10, 10, 2) * min(1.0, w / 640.0), _u(g, -tilt, tilt, 2)
        c, si = s * math.cos(th), s * math.sin(th)
        P = torch.tensor([[c, -si, float(t[0])], [si, c, float(t[1])], [float(p[0]), float(p[1]), 1.0]], dtype=torch.float64)
        off = torch.tensor([[1, 0, k * step + cx], [0, 1, cy], [0, 0, 1]], dtype=torch.float64)
        back = torch.tensor([[1, 0, -cx], [0, 1, -cy], [0, 0, 1]], dtype=torch.float64)
        H = off @ P @ back
        Hs.append(H / H[2, 2])
    pair = [torch.eye(3, dtype=torch.float64)]
    for k in range(1, n):
        H = torch.linalg.inv(Hs[k - 1]) @ Hs[k]
        pair.append(H / H[2, 2])
    canvas_w = n * step if case["ring"] else w + (n - 1) * step
    return dict(n_cams=n, W=w, H=h, ring=int(case["ring"]), ring_period=canvas_w if case["ring"] else 0,
                canvas_w=canvas_w, canvas_h=h, H_pair=[m.numpy() for m in pair], H_ref=Hs[0].numpy()), Hs


def _frames(case, rig, Hs, seed, steps=2):
    """`steps` consecutive frames of every camera: one texture, a smooth residual displacement the
    homographies do not describe, per-camera colour response, drifting exposure."""
    g = torch.Generator().manual_seed(seed)
    w, h, n = case["w"], case["h"], case["cams"]
    tex = _Texture(g, rig["canvas_w"], h, rig["ring_period"], 3)
    out = [[] for _ in range(steps)]
    us = torch.arange(w, device=DEV, dtype=torch.float64)
    for k in range(n):
        d = _smooth(g, w, h, 40, 3.0)
        M = torch.diag(_u(g, 0.8, 1.2, 3)) + _u(g, -0.05, 0.05, 3, 3) * (1 - torch.eye(3, dtype=torch.float64))
        M, gamma = M.float().to(DEV), float(_u(g, 0.9, 1.1, 1))
        gains = [1.0 + 0.01 * t * float(torch.randn(1, generator=g)) for t in range(steps)]
        H = Hs[k].tolist()
        fr = [torch.empty((h, w, 3), dtype=torch.uint8, device=DEV) for _ in range(steps)]
        for v0 in range(0, h, 1080):
            vs = torch.arange(v0, min(v0 + 1080, h), device=DEV, dtype=torch.float64)[:, None]
            den = H[2][0] * us + H[2][1] * vs + H[2][2]
            X = (H[0][0] * us + H[0][1] * vs + H[0][2]) / den + d[0, v0:v0 + len(vs)]
            Y = (H[1][0] * us + H[1][1] * vs + H[1][2]) / den + d[1, v0:v0 + len(vs)]
            if rig["ring_period"]:
                X = torch.remainder(X, float(rig["ring_period"]))
            rgb = tex(X.float(), Y.float())
            lin = sum(rgb[..., c:c + 1] * M[:, c] for c in range(3))
            for t in range(steps):
                fr[t][v0:v0 + len(vs)] = torch.floor(255.0 * (gains[t] * lin).clamp(0, 1) ** gamma + 0.5).to(torch.uint8)
        for t in range(steps):
            out[t].append(fr[t])
    return out


def _pair(g, w, h, reach):
    """(template, moving) luma, integer valued float32, and the planted displacement (2, h, w)"""
    tex = _Texture(g, w, h, 0, 1, rects=1 + int(torch.randint(0, 5, (1,), generator=g)))
    d = _smooth(g, w, h, 64, 0.5 + float(torch.rand(1, generator=g)) * (reach - 0.5))
    ys = torch.arange(h, device=DEV, dtype=torch.float32)[:, None].expand(h, w)
    xs = torch.arange(w, device=DEV, dtype=torch.float32)[None, :].expand(h, w)
    gain, off = float(_u(g, 0.97, 1.03, 1)), float(_u(g, -3, 3, 1))
    t, m = tex(xs, ys)[..., 0], tex(xs - d[0], ys - d[1])[..., 0]
    return torch.round(t * 255.0).contiguous(), torch.round(m * 255.0 * gain + off).clamp(0, 255).contiguous(), d


def _train_inputs(case, seed):
    """level-2 template / moving luma (n, h, w) and the label flow (n, h, w, 2) in level-2 px"""
    g = torch.Generator().manual_seed(seed)
    ts, ms, ls = [], [], []
    for _ in range(case["n"]):
        t, m, d = _pair(g, 4 * case["w"], 4 * case["h"], 8.0)
        ts.append(F.avg_pool2d(t[None, None], 4)[0, 0])
        ms.append(F.avg_pool2d(m[None, None], 4)[0, 0])
        ls.append(F.avg_pool2d(d[None], 4)[0].permute(1, 2, 0) / 4)
    return torch.stack(ts), torch.stack(ms), torch.stack(ls).contiguous()


def _conv_inputs(case, seed):
    """activations, weights and bias with the distributions of a trained layer; BF16 bits as int16"""
    g = torch.Generator(device=DEV).manual_seed(seed)
    P = case["n"] * case["w"] * case["h"]
    x = F.leaky_relu(torch.randn(P, case["cin"], device=DEV, generator=g), 0.1).bfloat16()
    wt = (torch.randn(case["cout"], 9, case["cin"], device=DEV, generator=g) * math.sqrt(2 / (9 * case["cin"]))).bfloat16()
    return x, wt, torch.randn(case["cout"], device=DEV, generator=g) * 0.05


def _stitcher(case, stream=0):
    rig, Hs = _rig(case, stream)
    st = V.Stitcher(rig, **(dict(flow=2) if case["flow"] == "variational" else {}))
    if case["flow"] == "surrogate":
        with open(WEIGHTS, "rb") as f:
            st.load_weights(f.read())
        st.set_flow_mode(V.FLOW_SURROGATE_FALLBACK, FB_TAU)
    return st, rig, Hs


def _streams(case):
    """3 and 4 cameras by turns, a larger size every second stream (16:9, 20 % overlap chains)"""
    out = []
    for i in range(case["streams"]):
        w = case["w"] + (i // 2) * case["step"]
        out.append(dict(cams=3 + i % 2, w=w, h=w * 9 // 16, overlap=0.20, ring=False, flow=case["flow"]))
    return out


def prepare(case, seed):
    kind = case["kind"]
    if kind == "stitch":
        st, rig, Hs = _stitcher(case)
        return dict(kind=kind, st=st, frames=_frames(case, rig, Hs, seed), pano=st.new_pano(DEV), t=0, state=case["state"])
    if kind == "batch":
        sts, frames = [], [[], []]
        for i, c in enumerate(_streams(case)):
            st, rig, Hs = _stitcher(c, stream=i)
            sts.append(st)
            for t, fr in enumerate(_frames(c, rig, Hs, seed + 1000003 * i)):
                frames[t].append(fr)
        return dict(kind=kind, batch=V.Batch(sts), frames=frames, panos=[st.new_pano(DEV) for st in sts], t=0)
    if kind == "flow":
        t, m, _ = _pair(torch.Generator().manual_seed(seed), case["w"], case["h"], 8.0)
        over = dict(flow=2) if case["flow"] == "variational" else {}
        return dict(kind=kind, pf=V.PlainFlow(case["w"], case["h"], **over), t=t, m=m)
    if kind == "train":
        t, m, lab = _train_inputs(case, seed)
        with open(WEIGHTS, "rb") as f:
            net = S.Net.from_blob(f.read(), max_pixels=max(1 << 19, t.numel()))
        return dict(kind=kind, net=net, t=t, m=m, lab=lab.reshape(-1, 2),
                    imgs=V.nn_images([(case["h"], case["w"])] * case["n"]))
    x, wt, b = _conv_inputs(case, seed)
    return dict(kind=kind, x=x.view(torch.int16), w=wt.view(torch.int16), b=b, cin=case["cin"], cout=case["cout"],
                imgs=V.nn_images([(case["h"], case["w"])] * case["n"]),
                mode=dict(lrelu=V.CONV_LRELU, linear=V.CONV_LINEAR, f32=V.CONV_F32)[case["mode"]])


def run(state):
    kind = state["kind"]
    if kind in ("stitch", "batch"):
        frames = state["frames"][state["t"]]
        state["t"] = (state["t"] + 1) % len(state["frames"])
        if kind == "batch":
            return state["batch"].run(frames, state["panos"])
        if state["state"]:
            pano, cs, _ = state["st"].stitch(frames, pano=state["pano"], want_state=True)
            return dict(pano=pano, state=torch.frombuffer(bytearray(V.state_bytes(cs)), dtype=torch.uint8))
        return state["st"].stitch(frames, pano=state["pano"])
    if kind == "flow":
        return state["pf"](state["t"], state["m"])
    if kind == "train":
        net = state["net"]
        pred = net.forward(S.pack(state["t"], state["m"]), state["imgs"])
        loss = net.backward(state["lab"])
        net.adam(lr=LR)
        params, grads = net.params()
        return dict(pred=pred, loss=loss, params=params, grads=grads)
    x, w, b = state["x"], state["w"], state["b"]
    f32 = state["mode"] == V.CONV_F32
    y = torch.empty((x.shape[0], state["cout"]), dtype=torch.float32 if f32 else torch.bfloat16, device=DEV)
    V.check(V.lib().vs_nn_conv3x3(C.c_void_p(x.data_ptr()), state["cin"], C.c_void_p(w.data_ptr()),
                                  C.c_void_p(b.data_ptr()), C.c_void_p(y.data_ptr()), state["cout"],
                                  C.byref(state["imgs"]), state["mode"], S.ALPHA,
                                  C.c_void_p(torch.cuda.current_stream().cuda_stream)), "vs_nn_conv3x3")
    return y


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

_LAYER_MACS = 9 * (2 * 32 + 3 * 32 * 32 + 32 * 2)   # per level-2 pixel: 2 live inputs, 2 live outputs


def _flow_flops(px, flow):
    """both directions over px level-0 pixels"""
    if flow == "surrogate":
        return 2 * px / 16 * 2 * _LAYER_MACS
    levels = 2 * px * 4 / 3
    # 12 flop per window tap and Gauss-Newton step; about 100 flop per pixel and Jacobi step (3 warps of 10)
    return levels * (12 * 81 * ITERS if flow == "plain" else 100 * 30)


def _stitch_work(c):
    step = int(round(c["w"] * (1.0 - c["overlap"])))
    canvas = (c["cams"] * step if c["ring"] else c["w"] + (c["cams"] - 1) * step) * c["h"]
    pairs = c["cams"] if c["ring"] else c["cams"] - 1
    return 3 * (c["cams"] * c["w"] * c["h"] + canvas), _flow_flops(pairs * c["overlap"] * c["w"] * c["h"], c["flow"])


def work(case):
    kind = case["kind"]
    if kind in ("stitch", "batch"):
        each = [_stitch_work(c) for c in (_streams(case) if kind == "batch" else [case])]
        return dict(bytes=sum(b for b, _ in each), flops=sum(f for _, f in each))
    px = case["w"] * case["h"] * case.get("n", 1)
    if kind == "flow":
        return dict(bytes=px * (2 * 4 + 2 * 8), flops=_flow_flops(px, case["flow"]))
    if kind == "train":
        # luma pair and label in, prediction and parameters out; forward, data and weight gradients
        return dict(bytes=px * (8 + 8 + 64) + 4 * 3 * 2 * 29000, flops=3 * 2 * px * _LAYER_MACS)
    return dict(bytes=px * 2 * (case["cin"] + case["cout"] * (2 if case["mode"] == "f32" else 1)),
                flops=2 * 9 * case["cin"] * case["cout"] * px)


# ---------------------------------------------------------------------------
# The same results in 64 bits, with plain torch
# ---------------------------------------------------------------------------

def exact(case, seed):
    kind = case["kind"]
    if kind == "flow" and case["flow"] == "plain":
        t, m, _ = _pair(torch.Generator().manual_seed(seed), case["w"], case["h"], 8.0)
        a, b = _pyramid(t.double()), _pyramid(m.double())
        return _lk(a, b), _lk(b, a)
    if kind == "train":
        return _train_exact(case, seed)
    if kind == "conv":
        x, wt, b = _conv_inputs(case, seed)
        y = torch.cat([_conv(xi.double(), wt.double(), case["h"], case["w"]) + b.double()
                       for xi in x.view(case["n"], -1, case["cin"])])
        return F.leaky_relu(y, S.ALPHA) if case["mode"] == "lrelu" else y
    return None   # panoramas are bytes; a state is whole numbers; the variational flow takes too long here


def _at(img, y, x):
    h, w = img.shape
    return img[y.clamp(0, h - 1), x.clamp(0, w - 1)]


def _pyramid(img):
    out = [img]
    for _ in range(LEVELS - 1):
        for dim in (1, 0):
            n = img.shape[dim]
            c = 2 * torch.arange((n + 1) // 2, device=img.device)
            img = sum(k * img.index_select(dim, (c + o).clamp(0, n - 1))
                      for o, k in zip(range(-2, 3), (1, 4, 6, 4, 1))) / 16
        out.append(img)
    return out


def _lk(T, M):
    """pyramidal Lucas-Kanade, P_M(x + f) ~ P_T(x), over the whole image: (h, w, 2)"""
    u = None
    for l in reversed(range(LEVELS)):
        t, m = T[l], M[l]
        h, w = t.shape
        y, x = torch.meshgrid(torch.arange(h, device=t.device), torch.arange(w, device=t.device), indexing="ij")
        gx, gy = 0.5 * (_at(t, y, x + 1) - _at(t, y, x - 1)), 0.5 * (_at(t, y + 1, x) - _at(t, y - 1, x))
        if u is None:
            u = [torch.zeros_like(t), torch.zeros_like(t)]
        else:
            hc, wc = u[0].shape
            cx, cy = (x * 0.5 - 0.25).clamp(0, wc - 1), (y * 0.5 - 0.25).clamp(0, hc - 1)
            xa, ya = cx.floor().long(), cy.floor().long()
            fx, fy = cx - xa, cy - ya
            u = [2 * ((1 - fy) * ((1 - fx) * _at(c, ya, xa) + fx * _at(c, ya, xa + 1))
                      + fy * ((1 - fx) * _at(c, ya + 1, xa) + fx * _at(c, ya + 1, xa + 1))) for c in u]
        taps = [(dy, dx) for dy in range(-RADIUS, RADIUS + 1) for dx in range(-RADIUS, RADIUS + 1)]
        G = [torch.zeros_like(t) for _ in range(3)]
        cnt = torch.zeros_like(t)
        for dy, dx in taps:
            ok = ((y + dy >= 0) & (y + dy < h) & (x + dx >= 0) & (x + dx < w)).double()
            a, b = _at(gx, y + dy, x + dx) * ok, _at(gy, y + dy, x + dx) * ok
            G[0], G[1], G[2], cnt = G[0] + a * a, G[1] + a * b, G[2] + b * b, cnt + ok
        g00, g01, g11 = G[0] + LAMBDA * cnt, G[1], G[2] + LAMBDA * cnt
        det = g00 * g11 - g01 * g01
        for _ in range(ITERS):
            ox, oy = u[0].floor(), u[1].floor()
            fx, fy = u[0] - ox, u[1] - oy
            ox, oy = ox.long(), oy.long()
            bu, bv = torch.zeros_like(t), torch.zeros_like(t)
            for dy, dx in taps:
                Y, X = y + dy, x + dx
                ok = ((Y >= 0) & (Y < h) & (X >= 0) & (X < w)).double()
                s = ((1 - fy) * ((1 - fx) * _at(m, Y + oy, X + ox) + fx * _at(m, Y + oy, X + ox + 1))
                     + fy * ((1 - fx) * _at(m, Y + oy + 1, X + ox) + fx * _at(m, Y + oy + 1, X + ox + 1)))
                e = (s - _at(t, Y, X)) * ok
                bu, bv = bu + _at(gx, Y, X) * e, bv + _at(gy, Y, X) * e
            u = [u[0] + (g01 * bv - g11 * bu) / det, u[1] + (g01 * bu - g00 * bv) / det]
    return torch.stack(u, dim=-1)


def _conv(x, wt, h, w):
    """zero-padded 3x3 cross-correlation of one image: x (h w, cin), wt (cout, 9, cin) -> (h w, cout)"""
    p = F.pad(x.view(h, w, -1), (0, 0, 1, 1, 1, 1))
    return sum(p[t // 3:t // 3 + h, t % 3:t % 3 + w].reshape(h * w, -1) @ wt[:, t].t().contiguous() for t in range(9))


def _train_exact(case, seed):
    T, M, lab = _train_inputs(case, seed)
    with open(WEIGHTS, "rb") as f:
        blob = f.read()
    n_layers, alpha = struct.unpack_from("<If", blob, 8)
    dims = [struct.unpack_from("<II", blob, 16 + 8 * i) for i in range(n_layers)]
    at, layers = 16 + 8 * n_layers, []
    for ci, co in dims:
        w = torch.frombuffer(bytearray(blob[at:at + 18 * ci * co]), dtype=torch.bfloat16).view(co, 9, ci)
        at += 18 * ci * co
        b = torch.frombuffer(bytearray(blob[at:at + 4 * co]), dtype=torch.float32)
        at += 4 * co
        layers.append((w.double().to(DEV).requires_grad_(), b.double().to(DEV).requires_grad_()))
    h, w = case["h"], case["w"]
    P = case["n"] * h * w
    preds, loss = [], torch.zeros((), dtype=torch.float64, device=DEV)
    for i in range(case["n"]):
        x = torch.zeros(h * w, 16, dtype=torch.float64, device=DEV)
        x[:, 0], x[:, 1] = (T[i].reshape(-1).double() - 128) / 64, (M[i].reshape(-1).double() - 128) / 64
        for j, (wt, b) in enumerate(layers):
            x = _conv(x, wt, h, w) + b
            x = F.leaky_relu(x, alpha) if j + 1 < n_layers else x
        e = ((x[:, :2] - lab[i].reshape(-1, 2).double()) ** 2).sum(1)
        part = torch.sqrt(e + 1e-6).sum()
        (part / P).backward()
        loss = loss + part.detach()
        preds.append(x.detach())
    params = torch.cat([q.detach().reshape(-1) for wb in layers for q in wb])
    grads = torch.cat([q.grad.reshape(-1) for wb in layers for q in wb])
    # the first Adam step: the moments divided by their bias corrections are g and g^2
    params = params - LR * grads / (grads.abs() + 1e-8)
    return dict(pred=torch.cat(preds), loss=loss, params=params, grads=grads)
