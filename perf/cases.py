"""The work that users of liblogfx have it do, as measurable cases.

listed() names the cases, draw() makes more of the same ranges, prepare()
builds what a user's program holds before the call (device images, a
context, parameters), run() is one pass through the public entry points,
work() what a pass cannot do without, and exact() the computed numbers in 64
bits from plain torch and numpy.

Images are synthetic scenes on the GPU: a gradient, axis-aligned rectangles
and thin polylines at the density of the package's 8192^2 scene, Gaussian
noise and salt-and-pepper impulses.
"""
import math
import os

import numpy as np
import torch

from paper_1304_3992_amd import logfx, scenes

DEV = "cuda"
HERE = os.path.dirname(os.path.abspath(logfx.__file__))
DEFAULT_MASKS = "5,0.8,9,1.4"          # the benchmark's pair of eq. (1) masks


def _single(name, h, w, bits, **kw):
    c = dict(name=name, kind="scene", h=h, w=w, bits=bits, smooth="always", median=5, cascade="",
             std5=-1.0, masks=DEFAULT_MASKS, grid=16, report=False)
    c.update(kw)
    return c


def listed():
    return [
        # a chip cut around a point of interest: the smallest calls, launches and host time count
        _single("chip_131x257_u8", 131, 257, 8, smooth="never"),
        # the package's 512 x 512 8-bit image: latency of one ordinary small call
        _single("image_512_u8", 512, 512, 8),
        # a 12-bit AWiFS-sized scene (2000^2), with the report a caller reads the thresholds from
        _single("scene_2000_u12_report", 2000, 2000, 12, report=True),
        # a Cartosat-sized panchromatic scene (4000^2, 8 bits), median applied in levels 5, 3, 5
        _single("scene_4000_u8_cascade", 4000, 4000, 8, cascade="3,5"),
        # the paper's two-stage deviation rule on a ragged 11-bit scene, unsmoothed
        _single("scene_3001x5003_u11_std5", 3001, 5003, 11, smooth="never", std5=20.0),
        # full-depth 16-bit pixels (bits left at the type's width), odd sides, 3 x 3 median
        _single("scene_6001x3501_u16", 6001, 3501, 16, median=3),
        # the headline scene: 8192^2, 11 bits, 5 x 5 median
        _single("scene_8192_u11", 8192, 8192, 11),
        # 64 uneven tiles (sides 256 .. 4096, 8-bit values in 16-bit words) in one batch call
        dict(name="batch_64_uneven", kind="batch", n=64, lo=256, hi=4096, shapes=3, bits=8, smooth="always"),
        # tiles of a multispectral scene, the trained gate deciding the median per tile
        dict(name="gated_32x2048_u11", kind="batch", n=32, lo=2048, hi=2048, shapes=0, bits=11, smooth="gate"),
        # one seamless scene, the gate deciding per region
        dict(name="regions_4096x8192_u11", kind="regions", rows=4, cols=8, region=1024, bits=11),
        # one training step's gradient of the gate at the trainer's batch size
        dict(name="gate_gradient_256", kind="gradient", batch=256, samples=1024),
        # logits of a validation batch
        dict(name="gate_logits_256", kind="logits", batch=256),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scene"] * 6 + ["batch", "batch", "regions", "gradient", "gradient", "logits"])
    if kind == "scene":
        h, w = _log_int(rng, 64, 8192), _log_int(rng, 64, 8192)
        bits = rng.choice([8, 8, 11, 11, 12, 16])
        extra = rng.choice(["", "", "", "cascade", "std5", "masks"])
        c = _single("", h, w, bits, smooth=rng.choice(["always", "always", "never"]), median=rng.choice([3, 5, 5]),
                    report=rng.random() < 0.25)
        if extra == "cascade":
            c["smooth"], c["cascade"] = "always", rng.choice(["3", "5", "3,5", "5,3,3"])
        elif extra == "std5":
            c["std5"] = round(rng.uniform(5.0, 40.0), 2)
        elif extra == "masks":
            c["masks"] = rng.choice(["3,0.5,5,0.8", "5,0.8,7,1.1", "7,1.1,9,1.4"])
            c["grid"] = rng.choice([12, 16, 23]) if h * w <= 4096 * 4096 else 16
        del c["name"]
        return c
    if kind == "batch":
        if rng.random() < 0.5:
            side = _log_int(rng, 256, 2048)
            n = rng.randint(2, max(2, min(32, 32 * 2048 * 2048 // (side * side))))
            return dict(kind="batch", n=n, lo=side, hi=side, shapes=0, bits=11, smooth="gate")
        return dict(kind="batch", n=rng.randint(2, 40), lo=rng.randint(128, 300), hi=rng.randint(1000, 3000),
                    shapes=rng.randint(1, 1 << 20), bits=rng.choice([8, 11, 12]), smooth=rng.choice(["always", "never"]))
    if kind == "regions":
        return dict(kind="regions", rows=rng.choice([1, 2, 4]), cols=rng.choice([2, 4, 8]),
                    region=rng.randint(256, 1024), bits=rng.choice([8, 11]))
    if kind == "gradient":
        return dict(kind="gradient", batch=_log_int(rng, 8, 256), samples=512)
    return dict(kind="logits", batch=_log_int(rng, 1, 1024))


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFF)
    return g


def _scene(h, w, bits, seed, words=None, noise=None, density=None):
    """One synthetic band; noise (in units of the 8-bit range) and impulse
    density may be maps.  8-bit images are uint8 unless `words` asks for
    16-bit words; deeper ones are int16 holding 16-bit pixels."""
    rng = np.random.default_rng(seed)
    g = _generator(seed)
    maxv = (1 << bits) - 1
    th = rng.uniform(0.0, 2.0 * math.pi)
    y = torch.arange(h, dtype=torch.float32, device=DEV)[:, None] * math.sin(th)
    x = torch.arange(w, dtype=torch.float32, device=DEV)[None, :] * math.cos(th)
    img = y + x
    lo, hi = float(img.min()), float(img.max())
    img = (img - lo) * (80.0 / max(hi - lo, 1e-6)) + 60.0
    nr = max(2, round(20000 * h * w / float(8192 * 8192)))
    hs, ws = rng.integers(8, 65, nr), rng.integers(8, 65, nr)
    ys, xs = rng.integers(0, h, nr), rng.integers(0, w, nr)
    vs = rng.integers(150, 251, nr)
    for a, b, c, d, v in zip(ys.tolist(), xs.tolist(), hs.tolist(), ws.tolist(), vs.tolist()):
        img[a:a + c, b:b + d] = float(v)
    for _ in range(max(1, round(500 * h * w / float(8192 * 8192)))):   # polyline segments, 1 to 3 pixels wide
        p = rng.uniform(0.0, 1.0, 4)
        n = int(max(h, w))
        t = torch.linspace(0.0, 1.0, n, device=DEV)
        r = ((p[0] + (p[1] - p[0]) * t) * (h - 1)).round().long()
        c = ((p[2] + (p[3] - p[2]) * t) * (w - 1)).round().long()
        v = float(rng.integers(150, 251))
        for k in range(int(rng.integers(1, 4))):
            img[(r + k).clamp_(max=h - 1), c] = v
    img *= maxv / 255.0
    s = noise if noise is not None else (4.0 if bits == 8 else 1.5)
    img += torch.randn(img.shape, generator=g, device=DEV) * s * (maxv / 255.0)
    img.round_().clamp_(0, maxv)
    d = density if density is not None else (0.0 if bits == 8 else 0.05)
    u = torch.rand(img.shape, generator=g, device=DEV)
    img[u < d / 2] = 0.0
    img[(u >= d / 2) & (u < d)] = float(maxv)
    if bits == 8 and not words:
        return img.to(torch.uint8)
    return img.to(torch.int32).to(torch.int16)   # 16-bit pixels, kept by their bits


def _masks(case):
    s1, g1, s2, g2 = case["masks"].split(",")
    return (int(s1), float(g1)), (int(s2), float(g2))


SMOOTH = {"always": logfx.SMOOTH_ALWAYS, "never": logfx.SMOOTH_NEVER, "gate": logfx.SMOOTH_GATE}


def _default_taps():
    return logfx.make_log_mask(5, 0.8, 16)[0], logfx.make_log_mask(9, 1.4, 16)[0]


def _theta(seed):
    """He-uniform initial parameters, as the trainer starts from."""
    rng = np.random.default_rng(seed)
    parts = []
    for shape in [(16, 3, 3, 3), (16,), (32, 16, 3, 3), (32,), (32, 32, 3, 3), (32,), (32,), (1,)]:
        lim = math.sqrt(6.0 / (np.prod(shape[1:]) if len(shape) > 1 else 32))
        zero = len(shape) == 1 and len(parts) != 6
        parts.append(np.zeros(shape).ravel() if zero else rng.uniform(-lim, lim, size=shape).ravel())
    return np.concatenate(parts).astype(np.float32)


def _features(n, seed):
    """Gate features of n tiles: mean value per cell (gradient, rectangles
    and noise) and two crossing densities that follow the tile's noise."""
    g = _generator(seed + 77)
    kw = dict(generator=g, device=DEV)
    base = 0.25 + 0.3 * torch.rand((n, 1, 1), **kw) * torch.linspace(0, 1, 128, device=DEV)[None, :, None]
    blocks = torch.rand((n, 32, 32), **kw)
    blocks = torch.where(blocks > 0.8, 0.35 * torch.rand((n, 32, 32), **kw), torch.zeros_like(blocks))
    mean = base + blocks.repeat_interleave(4, 1).repeat_interleave(4, 2) + 0.01 * torch.randn((n, 128, 128), **kw)
    level = torch.rand((n, 1, 1), **kw)
    d1 = 0.1 + 0.35 * level + 0.04 * torch.randn((n, 128, 128), **kw)
    d2 = 0.05 + 0.15 * level + 0.03 * torch.randn((n, 128, 128), **kw)
    return torch.stack([mean, d1, d2], 1).clamp_(0.0, 1.0).to(torch.bfloat16)


def _samples(case, seed):
    """Indices and labels of one training batch."""
    rng = np.random.default_rng(seed + 5)
    idx = rng.permutation(case["samples"])[:case["batch"]].astype(np.int32)
    labels = (rng.random(case["samples"]) < 0.5).astype(np.float32)
    return idx, labels


def _shapes(case):
    if case["lo"] == case["hi"]:
        return [(case["lo"], case["hi"])] * case["n"]
    return scenes.tile_shapes(case["n"], case["shapes"], case["lo"], case["hi"])


def prepare(case, seed):
    kind = case["kind"]
    ctx = logfx.Context(0)
    if kind == "scene":
        (s1, g1), (s2, g2) = _masks(case)
        cas = tuple(int(v) for v in case["cascade"].split(",") if v)
        params = logfx.Params(logfx.make_log_mask(s1, g1, case["grid"])[0], logfx.make_log_mask(s2, g2, case["grid"])[0],
                              smooth=SMOOTH[case["smooth"]], median_size=case["median"], median_cascade=cas,
                              std5_max=case["std5"])
        img = _scene(case["h"], case["w"], case["bits"], seed)
        return dict(kind=kind, ctx=ctx, params=params, img=img, bits=0 if case["bits"] in (8, 16) else case["bits"],
                    out=torch.empty(img.shape, dtype=torch.uint8, device=DEV), report=case["report"])
    if kind == "batch":
        params = logfx.Params(*_default_taps(), smooth=SMOOTH[case["smooth"]])
        rng = np.random.default_rng(seed + 9)
        imgs = []
        for i, (h, w) in enumerate(_shapes(case)):
            kw = {}
            if case["smooth"] == "gate":   # every tile has its own noise: the gate has real decisions to take
                sigma = float(rng.uniform(0.0, 2.5))
                kw = dict(noise=sigma, density=float(rng.uniform(0.0, 0.2)))
            imgs.append(_scene(h, w, case["bits"], seed + 1000 * (i + 1), words=True, **kw))
        if case["smooth"] == "gate":
            ctx.gate_load(os.path.join(HERE, "gate_weights.bin"))
        return dict(kind=kind, ctx=ctx, params=params, imgs=imgs, bits=case["bits"],
                    outs=[torch.empty(t.shape, dtype=torch.uint8, device=DEV) for t in imgs])
    if kind == "regions":
        r = case["region"]
        rng = np.random.default_rng(seed + 9)
        shape = (case["rows"], case["cols"])

        def spread(v):
            return torch.from_numpy(v.astype(np.float32)).to(DEV).repeat_interleave(r, 0).repeat_interleave(r, 1)

        img = _scene(r * shape[0], r * shape[1], case["bits"], seed, noise=spread(rng.uniform(0.0, 2.5, shape)),
                     density=spread(rng.uniform(0.0, 0.2, shape)))
        ctx.gate_load(os.path.join(HERE, "gate_weights.bin"))
        params = logfx.Params(*_default_taps(), smooth=logfx.SMOOTH_GATE, gate_region=r)
        return dict(kind=kind, ctx=ctx, params=params, img=img, bits=case["bits"],
                    out=torch.empty(img.shape, dtype=torch.uint8, device=DEV))
    ctx.gate_set_params(_theta(seed))
    if kind == "gradient":
        idx, labels = _samples(case, seed)
        return dict(kind=kind, ctx=ctx, feats=_features(case["samples"], seed), idx=torch.from_numpy(idx).to(DEV),
                    labels=torch.from_numpy(labels).to(DEV),
                    grad=torch.empty(logfx.GATE_NPARAM, dtype=torch.float32, device=DEV),
                    loss=torch.empty(1, dtype=torch.float32, device=DEV))
    return dict(kind=kind, ctx=ctx, feats=_features(case["batch"], seed),
                logits=torch.empty(case["batch"], dtype=torch.float32, device=DEV))


def run(state):
    kind, ctx = state["kind"], state["ctx"]
    if kind == "scene":
        return ctx.extract(state["img"], state["params"], state["out"], bits=state["bits"], report=state["report"])
    if kind == "batch":
        return ctx.extract_batch(state["imgs"], state["params"], state["outs"], bits=state["bits"])
    if kind == "regions":
        return ctx.extract(state["img"], state["params"], state["out"], bits=state["bits"])
    if kind == "gradient":
        return ctx.gate_backward(state["feats"], state["labels"], state["idx"], grad=state["grad"], loss=state["loss"])
    return ctx.gate_forward(state["feats"], logits=state["logits"])


# ------------------------------------------------------------------ work
NET_FORWARD = 2.0 * 9 * (16 * 3 * 64 * 64 + 32 * 16 * 32 * 32 + 32 * 32 * 16 * 16)   # per feature set
NET_BACKWARD = 2.0 * NET_FORWARD - 2.0 * 9 * 16 * 3 * 64 * 64   # weight gradients, and data gradients but the first


def work(case):
    kind = case["kind"]
    if kind == "scene":
        (s1, _), (s2, _) = _masks(case)
        px = case["h"] * case["w"]
        return {"bytes": px * ((1 if case["bits"] == 8 else 2) + 1), "flops": 2.0 * px * (s1 * s1 + s2 * s2)}
    if kind == "batch":
        px = sum(h * w for h, w in _shapes(case))
        net = NET_FORWARD * case["n"] if case["smooth"] == "gate" else 0.0
        return {"bytes": 3 * px, "flops": 2.0 * px * 106 + net}
    if kind == "regions":
        n = case["rows"] * case["cols"]
        px = n * case["region"] ** 2
        return {"bytes": px * ((1 if case["bits"] == 8 else 2) + 1), "flops": 2.0 * px * 106 + NET_FORWARD * n}
    feats = case["batch"] * 3 * 128 * 128 * 2
    if kind == "gradient":
        return {"bytes": feats + 2 * 4 * logfx.GATE_NPARAM, "flops": case["batch"] * (NET_FORWARD + NET_BACKWARD)}
    return {"bytes": feats + 4 * logfx.GATE_NPARAM + 4 * case["batch"], "flops": case["batch"] * NET_FORWARD}


# ------------------------------------------------------------------ exact
def _log_taps(size, sigma, grid):
    """eq. (1) sampled, its mean removed, rounded to the power-of-two grid,
    zero sum restored at the centre (64 bits)."""
    r = size // 2
    y, x = np.mgrid[-r:r + 1, -r:r + 1].astype(np.float64)
    q = (x * x + y * y) / (2.0 * sigma * sigma)
    v = -1.0 / (math.pi * sigma ** 4) * (1.0 - q) * np.exp(-q)
    v = v - v.sum() / v.size
    u = math.ldexp(1.0, math.frexp(float(np.abs(v).max()))[1] - grid)
    k = np.rint(v / u)
    k[r, r] -= k.sum()
    return k * u


def _sigma(img, taps):
    """Unbiased deviation of the crossing strengths of one mask."""
    r = taps.shape[0] // 2
    h, w = img.shape
    pad = torch.nn.functional.pad(img[None, None], (r, r, r, r), mode="replicate")[0, 0]
    L = torch.zeros_like(img)
    for i in range(2 * r + 1):
        for j in range(2 * r + 1):
            L += float(taps[i, j]) * pad[i:i + h, j:j + w]
    p = torch.nn.functional.pad(L[None, None], (1, 1, 1, 1), mode="replicate")[0, 0]
    up, dn, lf, rt = p[:-2, 1:-1], p[2:, 1:-1], p[1:-1, :-2], p[1:-1, 2:]
    hi = torch.maximum(torch.maximum(up, dn), torch.maximum(lf, rt))
    lo = torch.minimum(torch.minimum(up, dn), torch.minimum(lf, rt))
    cross = ((L < 0) & (L + hi >= 0)) | ((L > 0) & (L + lo < 0)) | ((L == 0) & ((lf * rt < 0) | (up * dn < 0)))
    z = torch.where(cross, torch.maximum(hi, L) - torch.minimum(lo, L), torch.zeros_like(L))
    return float(z.std())


def _network(theta, x):
    """The gate's logits in 64 bits; theta a flat float64 tensor."""
    at = 0

    def take(*shape):
        nonlocal at
        n = int(np.prod(shape))
        t = theta[at:at + n].reshape(shape)
        at += n
        return t

    for co, ci in ((16, 3), (32, 16), (32, 32)):
        w, b = take(co, ci, 3, 3), take(co)
        x = torch.relu(torch.nn.functional.conv2d(x, w, b, stride=2, padding=1))
    return x.mean((2, 3)) @ take(32) + take(1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "scene" and case["report"]:
        if case["h"] * case["w"] > 4096 * 4096:
            return None
        img = _scene(case["h"], case["w"], case["bits"], seed)
        img = (img.to(torch.int32) & 0xFFFF).to(torch.float64)
        sig = [_sigma(img, _log_taps(s, g, case["grid"])) for s, g in _masks(case)]
        return [None, {"sigma_g": sig, "thresh": [2.0 * s for s in sig]}]
    if kind == "gradient":
        idx, labels = _samples(case, seed)
        theta = torch.from_numpy(_theta(seed)).double().requires_grad_(True)
        x = _features(case["samples"], seed).cpu()[torch.from_numpy(idx).long()].double()
        y = torch.from_numpy(labels)[torch.from_numpy(idx).long()].double()
        loss = torch.nn.functional.binary_cross_entropy_with_logits(_network(theta, x), y)
        loss.backward()
        return [theta.grad, loss.detach().reshape(1)]
    if kind == "logits":
        with torch.no_grad():
            return _network(torch.from_numpy(_theta(seed)).double(), _features(case["batch"], seed).cpu().double())
    return None   # maps of 0 and 1 alone
