"""The work a user of this library has it do, as timed cases.

Kinds of case (the "kind" of a case dict), each through the public binding:

  code     images to first-spike times: DoG bank + rank-order coding in one
           call, the front of every image network;
  layer    one firing conv layer (optionally pooling its input first, or fed
           by a spike list): conv + fire, and when "learn" is set the layer's
           training half: lateral inhibition + k-WTA + STDP;
  readout  the last layer of a classifier (infinite threshold): pooling, conv,
           winner by potential, and when "learn" is set R-STDP from labels;
  fc       a fully connected layer: fire, winners, STDP;
  rate     one rate-coded layer: rate coding, integrate-and-fire with reset,
           rate pooling, firing rates;
  net      a whole call of a shipped workload: the three-layer net's training
           step, or the rate-coded network's inference.

Learning cases update a copy of the layer's weights, made in the pass, so every
pass (and every repeat of it) trains from the same weights: a run of
thousands of updates on one batch would drive them to their bounds, which no
training does.
"""
from __future__ import annotations

import dataclasses
import math

import torch

from paper_2301_13659_amd import pipeline, spk
from paper_2301_13659_amd import workloads as wls

DEV = "cuda"
NEVER = 255

# filter banks (kernel size, sigma1, sigma2), on-centre and off-centre pairs
BANKS = {
    "dog2": [(7, 1.0, 2.0), (7, 2.0, 1.0)],
    "dog6": [(3, 3 / 7, 6 / 7), (3, 6 / 7, 3 / 7), (7, 1.0, 2.0), (7, 2.0, 1.0),
             (13, 13 / 7, 26 / 7), (13, 26 / 7, 13 / 7)],
    "dog6x7": [(7, 0.5, 1.0), (7, 1.0, 0.5), (7, 1.0, 2.0), (7, 2.0, 1.0), (7, 1.5, 3.0), (7, 3.0, 1.5)],
}


# Master weights lie within 3e-5 of a multiple of 1/128 and thresholds halfway
# between two of its sums, so that no potential comes within rounding of a
# threshold: spike times are the same for every order of summation, while the
# weights' lower bits still have to be carried.
GRID = 128.0
HALF = 0.5 / GRID


def _layer(name, B, T, Ci, H, W, Co, K, stride, pad, theta, dtype, density, learn, k=5, radius=3,
           pool=0, pool_stride=0, pool_pad=0, source="spikes", spike_list=False, bank="dog6"):
    c = dict(kind="layer", B=B, T=T, Ci=Ci, H=H, W=W, Co=Co, K=K, stride=stride, pad=pad, theta=theta + HALF,
             dtype=dtype, density=density, learn=learn, k=k, radius=radius, pool=pool,
             pool_stride=pool_stride, pool_pad=pool_pad, source=source, spike_list=spike_list, bank=bank)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the input stage of the three-layer net at its batch: one small launch per step
        dict(name="code-28", kind="code", B=64, H=28, W=28, bank="dog6", T=15, image="strokes"),
        # the same stage on large images: over 8192 values per sample
        dict(name="code-160x250", kind="code", B=32, H=160, W=250, bank="dog6x7", T=30, image="edges"),
        # the smallest call: one layer on a batch of 8 small images, where launches count
        _layer("layer-small", 8, 15, 2, 28, 28, 32, 5, 1, 2, 15.0, "f32", 0.0, True, 5, 2,
               source="images", bank="dog2"),
        # the large-image net's first layer: few maps, many positions
        _layer("layer-few-maps", 32, 30, 6, 160, 250, 4, 5, 1, 2, 15.0, "f32", 0.0, True, 1, 0,
               source="images", bank="dog6x7"),
        # the three-layer net's second layer in training: dense pooled input, float masters
        _layer("layer-pooled", 64, 15, 30, 28, 28, 250, 3, 1, 1, 10.0, "f32", 0.45, True, 8, 1, 2, 2, 0),
        # the example network's second layer in inference: more channels than a wave holds weights for
        _layer("layer-deep", 64, 15, 100, 28, 28, 200, 3, 1, 1, 5.0, "f32", 0.3, False, 8, 1, 2, 2, 0),
        # the spike-input layer in training, the largest ordinary call
        _layer("layer-spikes", 128, 30, 64, 64, 64, 128, 3, 1, 1, 20.0, "f16", 0.05, True, 16, 2),
        # spikes that arrive as lists, odd sizes, float masters
        _layer("layer-list", 48, 20, 40, 57, 43, 75, 3, 1, 1, 8.0, "f32", 0.03, True, 8, 2,
               spike_list=True),
        # the R-STDP readout at its batch: 250 channels, 5x5, winner by potential, labels
        dict(name="readout-rstdp", kind="readout", B=256, T=15, Ci=250, H=14, W=14, Co=200, K=5, pad=2,
             pool=3, pool_stride=3, pool_pad=1, density=0.3, dtype="f32", learn=True),
        # a fully connected classifier layer in training
        dict(name="fc-train", kind="fc", B=256, T=15, I=1125, O=211, theta=60.0 + HALF, density=0.3, dtype="f32",
             k=4, radius=3),
        # whole calls: a training step of the three-layer net, and 300-step rate-coded inference
        dict(name="net-train", kind="net", workload=2, B=64),
        dict(name="net-rate", kind="net", workload=7, B=64),
    ]


# ------------------------------------------------------------------- drawing

def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _layer_cost(c):
    """Microseconds, roughly, at the rates these kernels reach."""
    Hi, Wi = _pooled(c)
    Ho, Wo = Hi + 2 * c["pad"] - c["K"] + 1, Wi + 2 * c["pad"] - c["K"] + 1
    fl = 2.0 * c["B"] * c["T"] * Ho * Wo * max(c["Co"], 32) * c["Ci"] * c["K"] ** 2
    rate = (4e8 if c["T"] <= 32 else 1e8) * (1.0 if c["dtype"] == "f16" else 0.5)
    return fl / rate + 5.0 * c["B"] * c["Co"] * Ho * Wo / 4e6


def _draw_layer(rng):
    style = rng.choice(["spikes", "spikes", "pooled", "images", "list"])
    while True:
        T = rng.choice([8, 10, 12, 15, 15, 15, 16, 20, 24, 30, 30, 32, 45, 60])
        learn = rng.random() < 0.5
        dtype = rng.choice(["f16", "f32"])
        k, radius = rng.randint(1, 16), rng.randint(0, 4)
        if style in ("spikes", "list"):
            K = rng.choice([3, 3, 3, 5])
            density = math.exp(rng.uniform(math.log(0.02), math.log(0.3 if style == "spikes" else 0.08)))
            Ci = _logint(rng, 8, 100)
            c = _layer(None, _logint(rng, 1, 128), T, Ci, _logint(rng, 12, 96), _logint(rng, 12, 96),
                       _logint(rng, 16, 200), K, 1, K // 2, 0.0, dtype, density, learn, k, radius,
                       spike_list=style == "list")
            fires = density
        elif style == "pooled":
            pool = rng.choice([2, 2, 3])
            density = rng.uniform(0.1, 0.5)
            c = _layer(None, _logint(rng, 4, 256), T, _logint(rng, 16, 128), _logint(rng, 20, 64),
                       _logint(rng, 20, 64), _logint(rng, 24, 300), 3, 1, 1, 0.0, dtype, density, learn, k,
                       radius, pool, pool, rng.choice([0, 0, 1]))
            fires = 1 - (1 - density) ** (pool * pool)
        else:
            bank = rng.choice(["dog2", "dog6", "dog6x7"])
            c = _layer(None, _logint(rng, 4, 128), T, len(BANKS[bank]), _logint(rng, 28, 200),
                       _logint(rng, 28, 200), _logint(rng, 4, 128), 5, 1, 2, 0.0, dtype, 0.0, learn, k,
                       radius, source="images", bank=bank)
            fires = 0.3
        # a threshold that part of the neurons reach, as training keeps it
        c["theta"] = HALF + max(1, round(0.8 * fires * c["Ci"] * c["K"] ** 2 * rng.uniform(0.3, 0.9)))
        if c["Ci"] * c["K"] ** 2 <= 1156 and _layer_cost(c) < 1200.0:
            return c


def draw(rng):
    kind = rng.choice(["layer"] * 6 + ["code", "readout", "fc", "rate"])
    if kind == "layer":
        return _draw_layer(rng)
    if kind == "code":
        while True:
            B, H, W = _logint(rng, 1, 256), _logint(rng, 20, 250), _logint(rng, 20, 250)
            if B * H * W <= 32 * 160 * 250:
                break
        return dict(kind="code", B=B, H=H, W=W, bank=rng.choice(sorted(BANKS)), T=rng.choice([8, 15, 20, 30, 60]),
                    image=rng.choice(["strokes", "edges"]))
    if kind == "readout":
        pool = rng.choice([2, 3])
        return dict(kind="readout", B=_logint(rng, 8, 256), T=rng.choice([15, 20, 30]), Ci=_logint(rng, 40, 256),
                    H=rng.randint(8, 15), W=rng.randint(8, 15), Co=_logint(rng, 20, 240), K=rng.choice([3, 5]),
                    pad=rng.choice([1, 2]), pool=pool, pool_stride=pool, pool_pad=rng.choice([0, 1]),
                    density=rng.uniform(0.1, 0.5), dtype=rng.choice(["f16", "f32"]), learn=rng.random() < 0.5)
    if kind == "fc":
        while True:
            B, T = _logint(rng, 8, 512), rng.choice([15, 20, 30])
            I, O = _logint(rng, 100, 4000), _logint(rng, 10, 1000)
            if B * T * I * O <= 256 * 15 * 1125 * 211:
                break
        density = rng.uniform(0.1, 0.6)
        return dict(kind="fc", B=B, T=T, I=I, O=O,
                    theta=HALF + max(1, round(0.8 * density * I * rng.uniform(0.2, 0.6))), density=density,
                    dtype=rng.choice(["f16", "f32"]), k=rng.randint(1, 8), radius=rng.randint(0, 4))
    while True:
        c = dict(kind="rate", B=_logint(rng, 4, 64), T=_logint(rng, 50, 400), Ci=rng.choice([2, 6, 25, 40]),
                 H=_logint(rng, 10, 40), W=_logint(rng, 10, 40), Co=_logint(rng, 10, 64), K=rng.choice([3, 5]),
                 theta=float(rng.randint(4, 20)), pool=rng.choice([2, 3]))
        px = c["B"] * c["T"] * c["H"] * c["W"]
        if px * (5 * c["Ci"] + 2 * c["Co"]) <= 8e8 and px * c["Co"] * c["Ci"] * c["K"] ** 2 <= 6e10:
            return c


# -------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEV)


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device=DEV)


def _band(n, sigma, radius):
    """n x n matrix of a zero-padded Gaussian blur along one axis (float64)."""
    d = torch.arange(n, device=DEV, dtype=torch.float64)
    d = d[:, None] - d[None, :]
    m = torch.exp(-d * d / (2 * sigma * sigma)) * (d.abs() <= radius)
    k = torch.arange(-radius, radius + 1, device=DEV, dtype=torch.float64)
    return m / torch.exp(-k * k / (2 * sigma * sigma)).sum()


def _segments(g, img, count, lo, hi, keep_max):
    """Draws `count` random line segments into each of the images B x H x W."""
    B, H, W = img.shape
    py = torch.arange(H, device=DEV)[:, None] + 0.5
    px = torch.arange(W, device=DEV)[None, :] + 0.5
    for _ in range(count):
        r = _rand(g, B, 6)
        y0, x0 = (r[:, 0] * H)[:, None, None], (r[:, 1] * W)[:, None, None]
        length = min(H, W) * (0.15 + 0.4 * r[:, 2])
        dy = (length * torch.sin(6.2832 * r[:, 3]))[:, None, None]
        dx = (length * torch.cos(6.2832 * r[:, 3]))[:, None, None]
        u = (((py - y0) * dy + (px - x0) * dx) / (dy * dy + dx * dx + 1e-6)).clamp(0, 1)
        d = torch.hypot(py - (y0 + u * dy), px - (x0 + u * dx))
        on = d <= (0.5 + r[:, 4])[:, None, None]
        v = (lo + (hi - lo) * r[:, 5])[:, None, None] * on
        img = torch.maximum(img, v) if keep_max else img + v
    return img


def _images(g, B, H, W, kind):
    """uint8 B x 1 x H x W: digit-like strokes on black, or textured scenes with edges."""
    if kind == "strokes":
        img = _segments(g, torch.zeros((B, H, W), device=DEV), 8, 160.0, 255.0, True)
    else:
        gh, gw = _band(H, 6.0, 24).float(), _band(W, 6.0, 24).float()
        n = gh @ _randn(g, B, H, W) @ gw
        lo, hi = n.amin((1, 2), keepdim=True), n.amax((1, 2), keepdim=True)
        img = _segments(g, (n - lo) / (hi - lo + 1e-9) * 160.0, 7, 60.0, 95.0, False)
    return img.round().clamp(0, 255).to(torch.uint8)[:, None].contiguous()


def _rank_times(x, T):
    """First-spike times of values x (B x ...) by rank among the positive ones, descending."""
    B = x.shape[0]
    v = x.reshape(B, -1)
    live = v > 0.01
    order = torch.argsort(torch.where(live, -v, torch.full_like(v, math.inf)), dim=1, stable=True)
    rank = torch.empty_like(order)
    rank.scatter_(1, order, torch.arange(v.shape[1], device=DEV).expand_as(order))
    n = live.sum(1, keepdim=True).clamp(min=1)
    t = torch.where(live, rank * T // n, torch.full_like(rank, NEVER))
    return t.to(torch.uint8).reshape(x.shape).contiguous()


def _coded_images(g, B, H, W, T, bank):
    """Time maps a first layer sees: differences of Gaussians of strokes, rank-order coded."""
    img = _images(g, B, H, W, "strokes" if H * W < 4000 else "edges")[:, 0].double() / 255
    blur = {}
    for _, a, b in BANKS[bank]:
        for s in (a, b):
            if s not in blur:
                r = max(1, round(3 * s))
                blur[s] = _band(H, s, r) @ img @ _band(W, s, r)
    x = torch.stack([blur[a] - blur[b] for _, a, b in BANKS[bank]], 1)
    return _rank_times(x, T)


def _spike_times(g, shape, T, density):
    on = _rand(g, *shape) < density
    t = (_rand(g, *shape) * T).clamp(max=T - 1).to(torch.uint8)
    return torch.where(on, t, torch.full_like(t, NEVER))


def _weights(g, shape, dtype):
    """float32 masters, normal around 0.8 (see GRID), or half weights uniform on
    [0.7, 0.9] (multiples of 2^-11 below 1: their sums are exact in any order)."""
    if dtype == "f16":
        h = (0.7 + 0.2 * _rand(g, *shape)).half()
        return h.float(), h
    w = (GRID * (0.8 + 0.05 * _randn(g, *shape)).clamp(0.1, 0.99)).round() / GRID
    return w + 3e-5 * (2 * _rand(g, *shape) - 1), None


def _pooled(c):
    if not c.get("pool"):
        return c["H"], c["W"]
    f = lambda n: (n + 2 * c["pool_pad"] - c["pool"]) // c["pool_stride"] + 1  # noqa: E731
    return f(c["H"]), f(c["W"])


STDP = [(0.004, -0.003, 0.0, 1.0, 1)]
RSTDP = [(0.004, -0.003, 0.0, 1.0, 1), (-0.0005, 0.004, 0.0, 1.0, 1)]


def prepare(case, seed):
    c, g = case, _gen(seed)
    s = {"c": c}
    if c["kind"] == "code":
        s["img"] = _images(g, c["B"], c["H"], c["W"], c["image"])
    elif c["kind"] == "layer":
        if c["source"] == "images":
            s["x"] = _coded_images(g, c["B"], c["H"], c["W"], c["T"], c["bank"])
        else:
            s["x"] = _spike_times(g, (c["B"], c["Ci"], c["H"], c["W"]), c["T"], c["density"])
        s["w"], s["w16"] = _weights(g, (c["Co"], c["Ci"], c["K"], c["K"]), c["dtype"])
        if c["spike_list"]:
            # a list of the layer's capacity: a tenth of the inputs
            s["list"] = spk.spk_times_to_spikes(s["x"], c["T"], max(64, c["Ci"] * c["H"] * c["W"] // 10))
    elif c["kind"] == "readout":
        s["x"] = _spike_times(g, (c["B"], c["Ci"], c["H"], c["W"]), c["T"], c["density"])
        s["w"], s["w16"] = _weights(g, (c["Co"], c["Ci"], c["K"], c["K"]), c["dtype"])
        s["labels"] = (_rand(g, c["B"]) * 10).clamp(max=9).to(torch.int32)
        s["group"] = max(1, -(-c["Co"] // 10))
        # a layer that does not learn has its weights packed once
        s["packed"] = None if c["learn"] else spk.spk_conv_pack_weights(s["w"] if s["w16"] is None else s["w16"])
    elif c["kind"] == "fc":
        s["x"] = _spike_times(g, (c["B"], c["I"]), c["T"], c["density"])
        s["w"], s["w16"] = _weights(g, (c["O"], c["I"]), c["dtype"])
    elif c["kind"] == "rate":
        blobs = _rand(g, c["B"], c["Ci"], c["H"], c["W"])
        s["x"] = (blobs * blobs * (_rand(g, c["B"], c["Ci"], c["H"], c["W"]) < 0.5)).contiguous()
        s["u"] = _rand(g, c["B"], c["T"], c["Ci"], c["H"], c["W"])
        s["w"] = (_rand(g, c["Co"], c["Ci"], c["K"], c["K"]) < 0.5).half()
    else:
        wl = wls.get(c["workload"])
        make = pipeline.RatePipeline if wl.coding == "rate" else pipeline.Pipeline
        s["pipe"] = p = make(wl.with_batch(1), DEV)
        p.wl = wl.with_batch(c["B"])
        p.images = _images(g, c["B"], *wl.image_hw, "strokes")
        if wl.coding == "rate":
            p.draws = _rand(g, c["B"], wl.T, *wl.input_chw())
        for layer, spec in zip(p.layers, wl.convs):
            w = (spec.w_mean + spec.w_std * _randn(g, *layer.w.shape)).clamp(0, 1)
            if wl.binarize is not None:
                w = (w >= wl.binarize).float()
            layer.w.copy_(w)
            if layer.w16 is not None:
                layer.w16.copy_(w)
            layer.repack()
        s["w0"] = [layer.w.clone() for layer in p.layers]
    return s


# --------------------------------------------------------------------- passes

def _train(out, w, w16, x, tf, vk, T, k, radius, cfgs, stride, pad, readout=False, labels=None, group=0):
    win, n = spk.spk_inhibit_winners(tf, vk, T, k, radius, pointwise=not readout, readout=readout)
    wc = None if labels is None else spk.spk_rstdp_select(win, n, labels, group)
    w1 = w.clone()
    h1 = None if w16 is None else w16.clone()
    spk.spk_stdp_update(w1, x, win, n, cfgs, stride, pad, winner_cfg=wc, w_f16=h1)
    out.update(winners=win[..., :4], v=win[..., 4].view(torch.float32), n=n, w=w1, w16=h1)


def run(state):
    s, c = state, state["c"]
    kind = c["kind"]
    if kind == "code":
        return spk.spk_dog_latency_code(s["img"], BANKS[c["bank"]], c["T"], 0.01)
    if kind == "layer":
        w_op = s["w"] if s["w16"] is None else s["w16"]
        T, geo = c["T"], (c["stride"], c["pad"], c["theta"])
        if c["spike_list"]:
            sp, off = s["list"]
            shape = (c["Ci"], c["H"], c["W"])
            tf, vk = spk.spk_conv_fire_sparse(sp, off, shape, w_op, T, *geo)
            x = spk.spk_spikes_to_times(sp, off, shape, T) if c["learn"] else None
        elif c["pool"]:
            r = spk.spk_pool_conv_fire(s["x"], (c["pool"], c["pool_stride"], c["pool_pad"]), w_op, T, *geo,
                                       keep_pooled=c["learn"])
            x, tf, vk = r if c["learn"] else (None,) + r
        else:
            x = s["x"]
            tf, vk = spk.spk_conv_fire(x, w_op, T, *geo)
        out = {"times": tf, "vkey": vk}
        if c["learn"]:
            _train(out, s["w"], s["w16"], x, tf, vk, T, c["k"], c["radius"], STDP, c["stride"], c["pad"])
        return out
    if kind == "readout":
        w_op = s["w"] if s["w16"] is None else s["w16"]
        r = spk.spk_pool_conv_fire(s["x"], (c["pool"], c["pool_stride"], c["pool_pad"]), w_op, c["T"], 1,
                                   c["pad"], math.inf, packed_w=s["packed"], keep_pooled=c["learn"])
        x, tf, vk = r if c["learn"] else (None,) + r
        out = {"vkey": vk}
        if c["learn"]:
            _train(out, s["w"], s["w16"], x, tf, vk, c["T"], 1, 0, RSTDP, 1, c["pad"], readout=True,
                   labels=s["labels"], group=s["group"])
        else:
            win, n = spk.spk_inhibit_winners(tf, vk, c["T"], 1, 0, pointwise=False, readout=True)
            out.update(winners=win[..., :4], v=win[..., 4].view(torch.float32), n=n)
        return out
    if kind == "fc":
        w_op = s["w"] if s["w16"] is None else s["w16"]
        tf, vk = spk.spk_fc_fire(s["x"], w_op, c["T"], c["theta"])
        win, n = spk.spk_fc_winners(tf, vk, c["T"], c["k"], c["radius"])
        w1 = s["w"].clone()
        h1 = None if s["w16"] is None else s["w16"].clone()
        spk.spk_fc_stdp_update(w1, s["x"], win, n, STDP, w_f16=h1)
        return {"times": tf, "vkey": vk, "winners": win[..., :4], "v": win[..., 4].view(torch.float32), "n": n,
                "w": w1, "w16": h1}
    if kind == "rate":
        f = spk.spk_rate_code(s["x"], s["u"], c["T"], 0.01)
        f, counts = spk.spk_conv_if_rate(f, s["w"], 1, c["K"] // 2, c["theta"])
        f, counts = spk.spk_rate_pool(f, counts, c["pool"])
        return {"frames": f, "counts": counts, "rates": spk.spk_rate_features(counts, c["T"])}
    p = s["pipe"]
    if p.wl.coding == "rate":
        o = p.step(keep=True)
        return {"rates": o.features, "counts": [counts for _, counts in o.layer_out],
                "frames": [f for f, _ in o.pooled]}
    for layer, w0 in zip(p.layers, s["w0"]):
        if layer.spec.stdp:
            layer.w.copy_(w0)
    o = p.step(keep=True)
    return {"times0": o.times0, "pooled": o.pooled, "times": [t for t, _ in o.layer_out[:-1]],
            "vkey": [v for _, v in o.layer_out],
            "winners": [o.winners[k][0][..., :4] for k in sorted(o.winners)],
            "w": [layer.w for layer in p.layers if layer.spec.stdp]}


# ------------------------------------------------------------- work and error

def _conv_work(B, Ci, Hi, Wi, Co, K, pad, spikes):
    """Bytes in and out of a firing layer (a byte per input, a time and a
    potential per neuron) and two operations per weight that an arriving spike adds."""
    Ho, Wo = Hi + 2 * pad - K + 1, Wi + 2 * pad - K + 1
    return B * Ci * Hi * Wi, 5.0 * B * Co * Ho * Wo, 2.0 * spikes * K * K * Co, B * Co * Ho * Wo


def work(case):
    c = case
    if c["kind"] == "code":
        px, F = c["B"] * c["H"] * c["W"], BANKS[c["bank"]]
        return {"bytes": px * (1.0 + len(F)), "flops": px * 2.0 * sum(k * k for k, _, _ in F)}
    if c["kind"] in ("layer", "readout"):
        Hi, Wi = _pooled(c)
        d = c["density"] or 0.4
        fires = 1 - (1 - d) ** (c["pool"] ** 2) if c["pool"] else d
        wsize = c["Co"] * c["Ci"] * c["K"] ** 2
        i, o, f, neurons = _conv_work(c["B"], c["Ci"], Hi, Wi, c["Co"], c["K"], c["pad"],
                                      fires * c["B"] * c["Ci"] * Hi * Wi)
        if c["kind"] == "readout":
            o = 4.0 * neurons
        i = c["B"] * c["Ci"] * c["H"] * c["W"]
        if c.get("spike_list"):
            i *= 4 * d
        total = i + o + wsize * (2 if c["dtype"] == "f16" else 4)
        if c["learn"]:
            total += 8.0 * wsize + (c["B"] * c["Ci"] * Hi * Wi if c["pool"] or c.get("spike_list") else 0)
            f += neurons
        return {"bytes": total, "flops": f}
    if c["kind"] == "fc":
        n = c["O"] * c["I"]
        return {"bytes": c["B"] * (c["I"] + 5.0 * c["O"]) + n * (12 if c["dtype"] == "f32" else 12),
                "flops": 2.0 * c["density"] * c["B"] * n}
    if c["kind"] == "rate":
        px = c["B"] * c["T"] * c["H"] * c["W"]
        # draws in, pooled frames out; the spikes between the calls are the calls' own output
        return {"bytes": px * (4.0 * c["Ci"] + c["Ci"] + c["Co"] + c["Co"] / c["pool"] ** 2),
                "flops": px * 2.0 * 0.17 * c["Ci"] * c["Co"] * c["K"] ** 2}
    wl = wls.get(c["workload"])
    C, H, W = wl.input_chw()
    B, byt, fl = c["B"], 0.0, 0.0
    rate = wl.coding == "rate"
    steps = wl.T if rate else 1
    byt += B * H * W + B * C * H * W * steps * (5.0 if rate else 1.0)
    fl += B * H * W * 2.0 * (sum(f.ksize ** 2 for f in wl.dog) or 2 * len(wl.log_stds) * wl.log_ksize ** 2)
    for kind, p in wl.stages:
        if kind == "pool":
            H, W = (H + 2 * p.pad - p.k) // p.stride + 1, (W + 2 * p.pad - p.k) // p.stride + 1
            byt += B * C * H * W * steps
        elif kind == "conv":
            Ho, Wo = H + 2 * p.pad - p.k + 1, W + 2 * p.pad - p.k + 1
            fl += 2.0 * B * Ho * Wo * p.co * C * p.k ** 2 * (0.1 * steps if rate else 0.5)
            byt += B * p.co * Ho * Wo * (1.0 * steps if rate else 5.0) + p.co * C * p.k ** 2 * 4.0
            C, H, W = p.co, Ho, Wo
    return {"bytes": byt, "flops": fl}


def tolerance(case):
    """Potentials and weights to the rounding of 32-bit sums.  Winners are ranked
    by potential: two within rounding of each other may swap, and the update of
    the weights follows them.  In a whole network a potential within rounding
    of its threshold moves a spike, which later layers see."""
    c = case
    if c["kind"] in ("code", "rate") or (c["kind"] == "net" and wls.get(c["workload"]).coding == "rate"):
        return "exact"  # whole numbers; binary weights sum exactly
    if c["kind"] == "net":
        return {"rel": 1e-3, "max": 0.9, "differ": 2e-3}
    if c["dtype"] == "f16" and c["kind"] != "readout":
        return {"rel": 5e-5, "max": 1e-3, "differ": 0.0}  # exact potentials; updated weights round
    return {"rel": 2e-4, "max": 0.3, "differ": 4e-3}


# --------------------------------------------------------- 64-bit references

def _pool64(x, c):
    if not c.get("pool"):
        return x
    p = c["pool_pad"]
    v = torch.nn.functional.pad(x.double(), (p, p, p, p), value=float(NEVER))
    return v.unfold(2, c["pool"], c["pool_stride"]).unfold(3, c["pool"], c["pool_stride"]).amin((4, 5)).to(torch.uint8)


def _patches(x, K, pad):
    """uint8 B x Ci x H x W -> B x Ci*K*K x L windows (padding never fires)."""
    v = torch.nn.functional.pad(x.to(torch.float32), (pad,) * 4, value=float(NEVER))
    v = v.unfold(2, K, 1).unfold(3, K, 1)  # B Ci Ho Wo K K
    B, Ci, Ho, Wo = v.shape[:4]
    return v.permute(0, 1, 4, 5, 2, 3).reshape(B, Ci * K * K, Ho * Wo).to(torch.uint8), Ho, Wo


def _fire64(x, w, T, K, pad, theta):
    """(times, v_key) in 64 bits: the potential step by step, the first crossing of theta."""
    B, Co = x.shape[0], w.shape[0]
    wm = w.double().reshape(Co, -1)
    times, keys = [], []
    chunk = max(1, int(1.5e8 // max(1, wm.shape[1] * x.shape[2] * x.shape[3])))
    for b0 in range(0, B, chunk):
        pt, Ho, Wo = _patches(x[b0:b0 + chunk], K, pad)
        n, k, L = pt.shape
        pt = pt.permute(1, 0, 2).reshape(k, n * L)
        tf = torch.full((Co, n * L), NEVER, dtype=torch.uint8, device=DEV)
        key = torch.zeros((Co, n * L), dtype=torch.float64, device=DEV)
        V = torch.zeros((Co, n * L), dtype=torch.float64, device=DEV)
        for t in ([T - 1] if math.isinf(theta) else range(T)):
            V = wm @ (pt <= t).double()
            open_ = tf == NEVER
            key = torch.where(open_, V, key)
            tf = torch.where(open_ & (V > theta), torch.full_like(tf, t), tf)
        times.append(tf.reshape(Co, n, Ho, Wo).transpose(0, 1))
        keys.append(key.reshape(Co, n, Ho, Wo).transpose(0, 1))
    return torch.cat(times).contiguous(), torch.cat(keys).contiguous()


def _order(tf, key, readout):
    """Position of every neuron (B x n) in the order (time, potential descending, index)."""
    n = tf.shape[1]
    o = torch.argsort(-key, dim=1, stable=True)
    if not readout:
        o = o.gather(1, torch.argsort(tf.gather(1, o).to(torch.int32), dim=1, stable=True))
    pos = torch.empty_like(o)
    pos.scatter_(1, o, torch.arange(n, device=DEV).expand_as(o))
    return pos


def _winners64(tf, key, T, k, radius, readout, line=False):
    """Greedy k winners: (c, y, x, t) int32 B x k x 4, potentials, counts."""
    B, C, H, W = tf.shape
    n = C * H * W
    pos = _order(tf.reshape(B, n), key.reshape(B, n), readout)
    live = torch.ones((B, n), dtype=torch.bool, device=DEV) if readout else tf.reshape(B, n) != NEVER
    if not readout and not line:  # one survivor per location
        p = torch.where(live, pos, n).reshape(B, C, H * W)
        live = (p == p.amin(1, keepdim=True)).reshape(B, n) & live
    idx = torch.arange(n, device=DEV)
    cc, yy, xx = idx // (H * W), idx // W % H, idx % W
    win = torch.zeros((B, k, 4), dtype=torch.int32, device=DEV)
    win[..., 0] = -1
    v = torch.zeros((B, k), dtype=torch.float64, device=DEV)
    num = torch.zeros(B, dtype=torch.int32, device=DEV)
    for j in range(k):
        best, at = torch.where(live, pos, n).min(1)
        ok = best < n
        t = torch.full_like(at, T - 1) if readout else tf.reshape(B, n).gather(1, at[:, None])[:, 0].long()
        rec = torch.stack([cc[at], yy[at], xx[at], t], 1).to(torch.int32)
        win[:, j] = torch.where(ok[:, None], rec, win[:, j])
        v[:, j] = torch.where(ok, key.reshape(B, n).gather(1, at[:, None])[:, 0], 0.0)
        num += ok.to(torch.int32)
        if line:
            gone = (cc[None] - cc[at][:, None]).abs() <= radius
        else:
            gone = (cc[None] == cc[at][:, None]) | (((yy[None] - yy[at][:, None]).abs() <= radius) &
                                                    ((xx[None] - xx[at][:, None]).abs() <= radius))
        live = live & ~(gone & ok[:, None])
    return win, v, num


def _stdp64(w, x, win, num, cfgs, pad, cfg_of=None):
    """w + the winners' summed changes, clamped (64 bits); w Co x Ci x K x K, x B x Ci x H x W."""
    w = w.double()
    K = w.shape[2]
    xp = torch.nn.functional.pad(x.float(), (pad,) * 4, value=float(NEVER))
    pt = xp.unfold(2, K, 1).unfold(3, K, 1)
    B, k = win.shape[:2]
    sel = (torch.arange(k, device=DEV)[None] < num[:, None]).nonzero()
    D = torch.zeros_like(w)
    for at in sel.split(256):
        b, j = at[:, 0], at[:, 1]
        c, y, xx, t = win[b, j].long().unbind(1)
        causal = pt[b, :, y, xx] <= t[:, None, None, None]
        cf = torch.zeros_like(b) if cfg_of is None else cfg_of[b, j].long()
        a = torch.tensor([[f[0], f[1]] for f in cfgs], dtype=torch.float32, device=DEV).double()[cf]
        rate = torch.where(causal, a[:, 0, None, None, None], a[:, 1, None, None, None])
        lo, up = cfgs[0][2], cfgs[0][3]
        D.index_add_(0, c, rate * (w[c] - lo) * (up - w[c]))
    return (w + D).clamp(cfgs[0][2], cfgs[0][3])


def exact(case, seed):
    c = case
    if c["kind"] not in ("layer", "readout", "fc"):
        return None  # whole numbers, or a whole network
    s = prepare(case, seed)
    w = s["w"] if s["w16"] is None else s["w16"].float()
    if c["kind"] == "fc":
        x = s["x"][:, :, None, None]
        tf, key = _fire64(x, w[:, :, None, None], c["T"], 1, 0, c["theta"])
        win, v, num = _winners64(tf, key, c["T"], c["k"], c["radius"], False, line=True)
        w1 = None
        if s["w16"] is not None:  # (float masters: winners within rounding of each other may swap)
            w1 = _stdp64(s["w"][:, :, None, None], x, win, num, STDP, 0)[:, :, 0, 0]
        return {"times": None, "vkey": key[:, :, 0, 0], "winners": None, "v": v, "n": None, "w": w1, "w16": w1}
    x = _pool64(s["x"], c)
    if c.get("spike_list"):
        sp, off = s["list"]
        if int(off[:, -1].max()) > sp.shape[1]:
            return None  # a list cut at its capacity
    readout = c["kind"] == "readout"
    tf, key = _fire64(x, w, c["T"], c["K"], c["pad"], math.inf if readout else c["theta"])
    out = {"vkey": key} if readout else {"times": None, "vkey": key}
    if c["learn"] or readout:
        k, r = (1, 0) if readout else (c["k"], c["radius"])
        win, v, num = _winners64(tf, key, c["T"], k, r, readout)
        out.update(winners=None, v=v, n=None)
    if c["learn"]:
        cfg = None
        if readout:
            cfg = (win[..., 0] // s["group"] != s["labels"][:, None]).long()
        w1 = _stdp64(s["w"], x, win, num, RSTDP if readout else STDP, c["pad"], cfg)
        out.update(w=w1, w16=None if s["w16"] is None else w1)
    return out
