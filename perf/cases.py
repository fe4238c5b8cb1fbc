"""Performance cases of the library: whole calls through its public entry
points, over the sizes, precisions and options that users run.

A case is a dict of plain values; its "kind" says which entry points a pass
goes through:

  forward   GlassNet.forward, one frame batch (fp32, bf16 or fp8_t)
  train     one training step, autograd.train_step_adam from uploaded weights
  grad      the autograd functions: forward, L1 loss, backward to dL/dw
  stream    object streaming: begin, one accumulate per object, finish
  spatial   the spatial networks' forward
  sr        the x2 super-sampling network's forward
  sr_grad   its weight gradient

Inputs are drawn on the GPU from the seed with the recipe of
paper_2405_19056_amd/synth.py (G-buffer, slots with per-pixel uniform active
counts, scene vector, Kaiming-uniform weights).
"""
import math

import torch

from paper_2405_19056_amd import autograd as gn_autograd
from paper_2405_19056_amd.glassnet import GlassNet

DEV = "cuda:0"
NG, NL, NS, NOUT, ALPHA = 14, 12, 16, 3, 9


def listed():
    return [
        # a preview or probe frame at the smallest configured size: one short
        # launch, where latency is everything
        dict(name="fwd_bf16_64sq_k2_w64", kind="forward", precision="bf16", width=64, n=1, h=64,
             w=64, k=2, pool="mean", pe=0),
        # the paper's training resolution rendered frame by frame
        dict(name="fwd_bf16_256sq_k4", kind="forward", precision="bf16", width=128, n=1, h=256,
             w=256, k=4, pool="mean", pe=0),
        # the headline frame: full resolution, eight transparent objects
        dict(name="fwd_bf16_512sq_k8", kind="forward", precision="bf16", width=128, n=1, h=512,
             w=512, k=8, pool="mean", pe=0),
        # the largest serving resolution in the fp8 form
        dict(name="fwd_fp8_576x1024_k6", kind="forward", precision="fp8_t", width=128, n=1, h=576,
             w=1024, k=6, pool="mean", pe=0),
        # encoded inputs and the sum pool on a ragged window (no multiple of a tile)
        dict(name="fwd_bf16_pe2_333x517_k5", kind="forward", precision="bf16", width=128, n=1,
             h=333, w=517, k=5, pool="sum", pe=2),
        # the full-precision render (validation frames, teachers, calibration)
        dict(name="fwd_fp32_256sq_k4", kind="forward", precision="fp32", width=128, n=1, h=256,
             w=256, k=4, pool="mean", pe=0),
        # the configured training step: 16 crops, forward, L1 + DSSIM, backward, Adam
        dict(name="train_bf16_16x128sq_k4", kind="train", precision="bf16", width=128, n=16, h=128,
             w=128, k=4, pool="mean"),
        # fine-tuning on one small crop through torch.autograd: launches count
        dict(name="grad_fp32_64sq_k2_w64", kind="grad", precision="fp32", width=64, n=1, h=64,
             w=64, k=2, pool="mean", pe=0),
        # a frame whose objects arrive one at a time
        dict(name="stream_bf16_512sq_k8", kind="stream", precision="bf16", width=128, n=1, h=512,
             w=512, k=8, pool="mean"),
        # the spatial (U-Net) networks at the training resolution
        dict(name="spatial_256sq_k4", kind="spatial", precision="bf16", width=128, n=1, h=256,
             w=256, k=4, pool="mean"),
        # super-sampling a rendered frame to the display resolution
        dict(name="sr_256_to_512", kind="sr", n=1, h=256, w=256),
        # training the super-sampling network: its weight gradient on a batch
        dict(name="sr_grad_16x128sq", kind="sr_grad", n=16, h=128, w=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "forward", "train", "grad", "stream",
                       "spatial", "sr", "sr_grad"])
    pool = rng.choice(["mean", "mean", "sum"])
    if kind == "forward":
        prec = rng.choice(["bf16", "bf16", "fp32", "fp8_t"])
        width = 128 if prec == "fp8_t" else rng.choice([64, 128, 128])
        most = 512 if prec == "fp32" else 640
        h, w = _log_int(rng, 40, most), _log_int(rng, 40, most)
        return dict(kind=kind, precision=prec, width=width, n=rng.choice([1, 1, 1, 2]) if h * w < 90000
                    else 1, h=h, w=w, k=rng.randint(1, 8), pool=pool,
                    pe=rng.choice([0, 0, 0, rng.randint(1, 4)]))
    if kind in ("train", "grad"):
        n, h, w = _log_int(rng, 1, 16), _log_int(rng, 40, 128), _log_int(rng, 40, 128)
        c = dict(kind=kind, precision="bf16" if kind == "train" else "fp32",
                 width=rng.choice([64, 128, 128]), n=n, h=h, w=w, k=rng.randint(1, 4), pool=pool)
        if kind == "grad":
            c["pe"] = rng.choice([0, 0, 0, rng.randint(1, 4)])
        return c
    if kind == "stream":
        return dict(kind=kind, precision=rng.choice(["bf16", "bf16", "fp8_t"]), width=128, n=1,
                    h=_log_int(rng, 64, 512), w=_log_int(rng, 64, 512), k=rng.randint(2, 8),
                    pool=pool)
    if kind == "spatial":
        return dict(kind=kind, precision="bf16", width=rng.choice([64, 128, 128]), n=1,
                    h=2 * _log_int(rng, 24, 192), w=2 * _log_int(rng, 24, 192),
                    k=rng.randint(1, 8), pool=pool)
    if kind == "sr":
        return dict(kind=kind, n=1, h=_log_int(rng, 32, 384), w=_log_int(rng, 32, 384))
    return dict(kind=kind, n=_log_int(rng, 1, 16), h=_log_int(rng, 32, 128),
                w=_log_int(rng, 32, 128))


# ---- networks' shapes ---------------------------------------------------------

def _mlp_shapes(W, pe=0):
    e = 1 + 2 * pe
    return [(W, (NG + NS) * e), (W, W), (W, W), (W, NL * e + W), (W, W), (W, W),
            (W, 2 * W), (W, W), (W, W), (W, W + 3), (W, W), (NOUT, W)]


def _spatial_shapes(W):
    return [(W, NG + NS, 3), (W, W, 3), (W, 2 * W, 3), (W, W, 1),
            (W, NL + W, 3), (W, W, 1), (W, W, 1),
            (W, 2 * W, 3), (W, W, 3), (W, 2 * W, 3), (W, W, 1),
            (W, W + 3, 3), (W, W, 3), (NOUT, W, 1)]


def _sr_shapes():
    return [(32, 17, 3), (32, 32, 3), (3, 32, 1)]


# ---- inputs -------------------------------------------------------------------

def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + salt)
    return g


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device=DEV) * (hi - lo) + lo


def _weights(shapes, seed):
    """Kaiming-uniform matrices, uniform biases, packed layer by layer."""
    g, parts = _gen(seed, 1), []
    for s in shapes:
        fan_in = s[1] * (s[2] ** 2 if len(s) == 3 else 1)
        wb, bb = math.sqrt(6.0 / fan_in), 1.0 / math.sqrt(fan_in)
        parts += [_uniform(g, (s[0] * fan_in,), -wb, wb), _uniform(g, (s[0],), -bb, bb)]
    return torch.cat(parts)


def _normals(g, shape, axis):
    v = torch.randn(shape, generator=g, device=DEV)
    return v / v.norm(dim=axis, keepdim=True).clamp_min(1e-20)


def _gbuf(g, n, h, w):
    x = torch.empty((n, NG, h, w), device=DEV)
    x[:, 0:3] = _uniform(g, (n, 3, h, w), -1, 1)
    x[:, 3:6] = _normals(g, (n, 3, h, w), 1)
    x[:, 6:10] = _uniform(g, (n, 4, h, w), 0, 1)
    x[:, 10] = (_uniform(g, (n, h, w), 0, 1) < 0.3).float()
    x[:, 11:14] = _uniform(g, (n, 3, h, w), 0, 2)
    return x


def _layers(g, n, k, h, w):
    x = torch.empty((n, k, NL, h, w), device=DEV)
    x[:, :, 0:3] = _uniform(g, (n, k, 3, h, w), -1, 1)
    x[:, :, 3:6] = _normals(g, (n, k, 3, h, w), 2)
    x[:, :, 6:9] = _uniform(g, (n, k, 3, h, w), 0, 1)
    x[:, :, 10] = _uniform(g, (n, k, h, w), 1, 2)
    x[:, :, 11] = _uniform(g, (n, k, h, w), 0, 1)
    # per pixel an active count in 0..k and a random subset of that size
    count = torch.randint(0, k + 1, (n, 1, h, w), generator=g, device=DEV)
    rank = torch.rand((n, k, h, w), generator=g, device=DEV).argsort(1).argsort(1)
    x[:, :, ALPHA] = torch.where(rank < count, 1.0 - _uniform(g, (n, k, h, w), 0, 1), 0.0)
    return x


def _frame(c, seed):
    g = _gen(seed, 2)
    return (_gbuf(g, c["n"], c["h"], c["w"]), _layers(g, c["n"], c["k"], c["h"], c["w"]),
            _uniform(g, (c["n"], NS), -1, 1))


def _sr_inputs(c, seed):
    g = _gen(seed, 2)
    return (_uniform(g, (c["n"], 3, c["h"], c["w"]), 0, 2), _gbuf(g, c["n"], 2 * c["h"], 2 * c["w"]),
            torch.randn((c["n"], 3, 2 * c["h"], 2 * c["w"]), generator=g, device=DEV))


def _target(c, seed):
    """A noisy reference image in the range of the direct light."""
    return _uniform(_gen(seed, 3), (c["n"], 3, c["h"], c["w"]), 0, 2)


# ---- state --------------------------------------------------------------------

def prepare(case, seed):
    c = dict(case)
    s = {"case": c}
    if c["kind"] in ("sr", "sr_grad"):
        s["net"] = GlassNet(None, 64, precision="fp32")
        s["w"] = _weights(_sr_shapes(), seed)
        s["lo"], s["g"], s["dy"] = _sr_inputs(c, seed)
        return s
    W, pe = c["width"], c.get("pe", 0)
    s["g"], s["L"], s["s"] = _frame(c, seed)
    if c["kind"] == "spatial":
        s["net"] = GlassNet(None, W, k_max=8, pool=c["pool"], precision="bf16")
        s["w"] = _weights(_spatial_shapes(W), seed)
        return s
    s["w"] = _weights(_mlp_shapes(W, pe), seed)
    net = s["net"] = GlassNet(s["w"].cpu().numpy(), W, k_max=8, pool=c["pool"],
                              precision=c["precision"], pe_levels=pe)
    if c["precision"] == "fp8_t":       # one calibration frame, as a renderer starts up
        g = _gen(7, 4)
        net.calibrate(_gbuf(g, 1, 64, 64), _layers(g, 1, 8, 64, 64), _uniform(g, (1, NS), -1, 1))
    if c["kind"] in ("train", "grad"):
        s["t"] = _target(c, seed)
    if c["kind"] == "train":
        s["adam"] = net.adam_state()
    if c["kind"] == "grad":
        s["w"].requires_grad_(True)
    if c["kind"] == "stream":
        s["objects"] = [s["L"][:, i:i + 1].contiguous() for i in range(c["k"])]
        s["state"] = net.stream_state(c["n"], c["h"], c["w"], device=DEV)
    return s


def run(s):
    c, net = s["case"], s["net"]
    kind = c["kind"]
    if kind == "forward":
        return net.forward(s["g"], s["L"], s["s"])
    if kind == "train":
        # the first step from uploaded weights and fresh moments
        net.set_weights(s["w"])
        s["adam"].zero_()
        losses, gw = gn_autograd.train_step_adam(net, s["g"], s["L"], s["s"], s["t"], s["adam"], 1)
        return {"losses": losses, "grad": gw, "adam": s["adam"]}
    if kind == "grad":
        y = gn_autograd.GlassNetFunction.apply(net, s["g"], s["L"], s["s"], s["w"])
        loss = gn_autograd.L1Function.apply(net, y, s["t"])
        grad, = torch.autograd.grad(loss, s["w"])
        return {"y": y.detach(), "loss": loss.detach(), "grad": grad}
    if kind == "stream":
        net.stream_begin(s["g"], s["s"], s["state"])
        for obj in s["objects"]:
            net.stream_accumulate(obj, s["state"])
        return net.stream_finish(s["g"], s["state"])
    if kind == "spatial":
        return net.spatial_forward(s["w"], s["g"], s["L"], s["s"])
    if kind == "sr":
        return net.sr_forward(s["w"], s["lo"], s["g"])
    return net.sr_backward(s["w"], s["lo"], s["g"], s["dy"])


# ---- the work of a pass -------------------------------------------------------

def work(case):
    c = case
    kind, n, h, w = c["kind"], c["n"], c["h"], c["w"]
    px = n * h * w
    if kind in ("sr", "sr_grad"):
        hi = 4 * px
        params = sum(o * i * k * k + o for o, i, k in _sr_shapes())
        conv1, conv2, head = 32 * 17 * 9, 32 * 32 * 9, 96
        fwd = 2 * hi * (conv1 + conv2 + head)
        data = 4 * (3 * px + NG * hi)
        if kind == "sr":
            return {"bytes": data + 4 * (3 * hi + params), "flops": fwd}
        # recompute, the weight gradients, and the transposes of the head and conv2
        return {"bytes": data + 4 * (3 * hi + 2 * params),
                "flops": 2 * fwd + 2 * hi * (conv2 + head)}
    W, k = c["width"], c["k"]
    inputs = 4 * (px * (NG + NL * k) + n * NS)
    if kind == "spatial":
        mul = 87.5 * W * W + 2 * k * W * W + 300 * W + 108 * k * W
        params = sum(o * i * q * q + o for o, i, q in _spatial_shapes(W))
        return {"bytes": inputs + 4 * (3 * px + params), "flops": 2 * px * mul}
    e = 1 + 2 * c.get("pe", 0)
    params = sum(o * i + o for o, i in _mlp_shapes(W, c.get("pe", 0)))
    # per pixel: F's and h's input layers, then W x W ones (h's sigma part and
    # its affine last layer once per pixel, its hidden layer once per slot)
    first = (NG + NS) * e * W + k * NL * e * W
    rest = (10 + k) * W * W + 2 * 3 * W
    fwd = 2 * px * (first + rest)
    if kind in ("forward", "stream"):
        return {"bytes": inputs + 4 * (3 * px + params), "flops": fwd}
    # forward, then the deltas of every layer but the input ones and the weight gradients
    total = 2 * fwd + 2 * px * rest
    moved = inputs + 4 * (2 * 3 * px + 2 * params)
    if kind == "train":
        return {"bytes": moved + 4 * 4 * params, "flops": total}
    return {"bytes": moved + 4 * 3 * px, "flops": total}


# ---- the same in 64 bits ------------------------------------------------------

def _unpack(w, shapes):
    w, out, at = w.detach().double(), [], 0
    for s in shapes:
        m = s[1] * (s[2] ** 2 if len(s) == 3 else 1)
        A = w[at:at + s[0] * m].reshape(s[0], m)
        at += s[0] * m
        out.append((A, w[at:at + s[0]]))
        at += s[0]
    return out


def _encode(x, pe):
    blocks = [x]
    for i in range(pe):
        blocks += [torch.sin(2 ** i * math.pi * x), torch.cos(2 ** i * math.pi * x)]
    return torch.cat(blocks, 1)


def _pooled(zs, act, pool):
    total = sum(z * a for z, a in zip(zs, act))
    return total if pool == "sum" else total / sum(act).clamp_min(1.0)


def _net64(P, G, L, S, pool, pe):
    """[P][14], [P][k][12], [P][16] -> [P][3], layer by layer."""
    def lin(i, x):
        return x @ P[i][0].t() + P[i][1]

    def mlp(i, x):
        return lin(i + 2, torch.relu(lin(i + 1, torch.relu(lin(i, x)))))
    sigma = mlp(0, _encode(torch.cat([G, S], 1), pe))
    slots = [mlp(3, torch.cat([_encode(L[:, i], pe), sigma], 1)) for i in range(L.shape[1])]
    act = [(L[:, i, ALPHA:ALPHA + 1] > 0).double() for i in range(L.shape[1])]
    phi = mlp(6, torch.cat([sigma, _pooled(slots, act, pool)], 1))
    return mlp(9, torch.cat([phi, G[:, 11:14]], 1))


def _columns(g, L, s):
    n, _, h, w = g.shape
    G = g.double().permute(0, 2, 3, 1).reshape(n * h * w, NG)
    Ls = L.double().permute(0, 3, 4, 1, 2).reshape(n * h * w, L.shape[1], NL)
    return G, Ls, s.double().repeat_interleave(h * w, 0)


def _image(y, c, ch=3):
    return y.reshape(c["n"], c["h"], c["w"], ch).permute(0, 3, 1, 2).contiguous()


def _forward64(c, P, g, L, s):
    G, Ls, S = _columns(g, L, s)
    step = 1 << 17
    return _image(torch.cat([_net64(P, G[i:i + step], Ls[i:i + step], S[i:i + step], c["pool"],
                                    c.get("pe", 0)) for i in range(0, G.shape[0], step)]), c)


def _conv64(x, layer, k):
    """x [n][h][w][C] -> [n][h][w][out]: k x k correlation, zero padding."""
    A, b = layer
    n, h, w, C = x.shape
    A = A.reshape(A.shape[0], C, k, k)
    r = k // 2
    p = torch.nn.functional.pad(x, (0, 0, r, r, r, r))
    y = b
    for dy in range(k):
        for dx in range(k):
            y = y + p[:, dy:dy + h, dx:dx + w] @ A[:, :, dy, dx].t()
    return y


def _spatial64(P, g, L, s, pool):
    n, _, h, w = g.shape

    def unet(i, x):
        e1 = torch.relu(_conv64(x, P[i], 3))
        d = e1.reshape(n, h // 2, 2, w // 2, 2, -1).mean((2, 4))
        m = torch.relu(_conv64(d, P[i + 1], 3))
        up = m.repeat_interleave(2, 1).repeat_interleave(2, 2)
        return _conv64(torch.relu(_conv64(torch.cat([e1, up], 3), P[i + 2], 3)), P[i + 3], 1)
    G = g.double().permute(0, 2, 3, 1)
    S = s.double()[:, None, None, :].expand(n, h, w, NS)
    sigma = unet(0, torch.cat([G, S], 3))
    zs, act = [], []
    for i in range(L.shape[1]):
        b = L[:, i].double().permute(0, 2, 3, 1)
        z = torch.relu(_conv64(torch.cat([b, sigma], 3), P[4], 3))
        zs.append(_conv64(torch.relu(_conv64(z, P[5], 1)), P[6], 1))
        act.append((b[..., ALPHA:ALPHA + 1] > 0).double())
    phi = unet(7, torch.cat([sigma, _pooled(zs, act, pool)], 3))
    r = torch.relu(_conv64(torch.cat([phi, G[..., 11:14]], 3), P[11], 3))
    y = _conv64(torch.relu(_conv64(r, P[12], 3)), P[13], 1)
    return y.permute(0, 3, 1, 2).contiguous()


def _upsample64(x):
    """Bilinear x2, half-pixel centres, sources clamped at the edges."""
    for d in (2, 3):
        m = x.shape[d]
        i = torch.arange(m, device=x.device)
        prev, nxt = x.index_select(d, (i - 1).clamp_min(0)), x.index_select(d, (i + 1).clamp_max(m - 1))
        pair = torch.stack([0.25 * prev + 0.75 * x, 0.75 * x + 0.25 * nxt], d + 1)
        x = pair.flatten(d, d + 1)
    return x


def _sr64(P, lo, g):
    up = _upsample64(lo.double())
    x = torch.cat([up, g.double()], 1).permute(0, 2, 3, 1)
    a = torch.relu(_conv64(torch.relu(_conv64(x, P[0], 3)), P[1], 3))
    return up + _conv64(a, P[2], 1).permute(0, 3, 1, 2)


def _dssim64(x, y):
    t = torch.arange(11, dtype=torch.float64, device=x.device) - 5
    k = torch.exp(-t * t / (2 * 1.5 ** 2))
    k = k / k.sum()

    def local(v):
        h, w = v.shape[2:]
        v = sum(k[i] * v[:, :, i:i + h - 10] for i in range(11))
        return sum(k[i] * v[:, :, :, i:i + w - 10] for i in range(11))
    mx, my, c1, c2 = local(x), local(y), 0.01 ** 2, 0.03 ** 2
    vx, vy, cov = local(x * x) - mx * mx, local(y * y) - my * my, local(x * y) - mx * my
    ssim = (2 * mx * my + c1) * (2 * cov + c2) / ((mx * mx + my * my + c1) * (vx + vy + c2))
    return (1 - ssim.mean()) / 2


def exact(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind in ("sr", "sr_grad"):
        P = _unpack(_weights(_sr_shapes(), seed), _sr_shapes())
        lo, g, dy = _sr_inputs(c, seed)
        if kind == "sr":
            return _sr64(P, lo, g)
        flat = [t.clone().requires_grad_(True) for layer in P for t in layer]
        y = _sr64(list(zip(flat[0::2], flat[1::2])), lo, g)
        return torch.cat([t.reshape(-1) for t in torch.autograd.grad((y * dy.double()).sum(), flat)])
    g, L, s = _frame(c, seed)
    W, pe = c["width"], c.get("pe", 0)
    if kind == "spatial":
        return _spatial64(_unpack(_weights(_spatial_shapes(W), seed), _spatial_shapes(W)), g, L, s,
                          c["pool"])
    shapes = _mlp_shapes(W, pe)
    P = _unpack(_weights(shapes, seed), shapes)
    if kind in ("forward", "stream"):
        return _forward64(c, P, g, L, s)
    t = _target(c, seed).double()
    if kind == "train":
        # the sign of y - t flips between a bf16 render and an exact one at a
        # visible share of the pixels: the gradient has no exact counterpart
        y = _forward64(c, P, g, L, s)
        return {"losses": torch.stack([(y - t).abs().mean(), _dssim64(y, t)]), "grad": None,
                "adam": None}
    flat = [v.clone().requires_grad_(True) for layer in P for v in layer]
    G, Ls, S = _columns(g, L, s)
    tc, count = t.permute(0, 2, 3, 1).reshape(-1, 3), t.numel()
    grads, ys, loss = [torch.zeros_like(v) for v in flat], [], 0.0
    step = 1 << 16
    for i in range(0, G.shape[0], step):
        y = _net64(list(zip(flat[0::2], flat[1::2])), G[i:i + step], Ls[i:i + step], S[i:i + step],
                   c["pool"], pe)
        part = (y - tc[i:i + step]).abs().sum() / count
        grads = [a + b for a, b in zip(grads, torch.autograd.grad(part, flat))]
        ys.append(y.detach())
        loss = loss + part.detach()
    return {"y": _image(torch.cat(ys), c), "loss": loss,
            "grad": torch.cat([v.reshape(-1) for v in grads])}
