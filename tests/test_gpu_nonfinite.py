"""Infinite, NaN and very large values in the fp32 kernels, whose operands are
split in bf16 parts: what comes out is infinite, NaN or finite where fp32
products and sums make it so (compared with 64 bits; a ReLU of NaN is 0, as
fmax has it), and finite values agree.
"""
import numpy as np
import pytest

from paper_2405_19056_amd import synth
from paper_2405_19056_amd.glassnet import GlassNet

from gpu_util import log, torch_dev
from ref64 import SR_SHAPES, columns, conv64, glassnet64, layers_of

pytestmark = pytest.mark.gpu

VALUES = {"inf": float("inf"), "-inf": -float("inf"), "nan": float("nan")}
H, WD, K = 24, 40, 3


def fmax0(x):
    torch = torch_dev()
    return torch.fmax(x, torch.zeros_like(x))


def compare(y, ref, what):
    """The same kind everywhere; finite values within 1e-5 of their norm (the
    fp32 forward's own error is below 1e-6)."""
    torch = torch_dev()
    y, ref = y.double(), ref.detach()
    for kind in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(kind(y), kind(ref)), (what, kind.__name__)
    m = torch.isfinite(ref)
    err = float((y[m] - ref[m]).norm() / ref[m].norm())
    log(f"  {what}: {int((~m).sum())} not finite, others relF {err:.1e}")
    assert err <= 1e-5, what


def frame(W):
    torch = torch_dev()
    gen = torch.Generator(device="cuda:0").manual_seed(W)
    r = lambda *s: torch.rand(s, generator=gen, device="cuda:0") * 2 - 1  # noqa: E731
    g, L, s = r(1, 14, H, WD), r(1, K, 12, H, WD), r(1, 16)
    L[0, :, 9, 5:9, 7:11] = 0.5                      # every slot active here,
    L[0, 1, 9, 15, 20] = 0.0                         # one not
    return synth.make_weights(W, np.random.default_rng(W)), g, L, s


@pytest.mark.parametrize("W", [64, 128])
@pytest.mark.parametrize("value", list(VALUES))
def test_fp32_forward_and_streaming(W, value):
    wts, g0, L0, s0 = frame(W)
    v = VALUES[value]
    flat = layers_of(wts, synth.layer_shapes(W))
    cases = {}
    for plane in (0, 6, 11, 13):                     # position, albedo, L_d
        g = g0.clone()
        g[0, plane, 6, 8] = v
        cases[f"G-buffer plane {plane}"] = (g, L0, s0)
    for what, ch, y, x in (("active", 2, 6, 9), ("active", 11, 7, 8), ("inactive", 7, 15, 20)):
        L = L0.clone()
        L[0, 1, ch, y, x] = v
        cases[f"{what} slot, channel {ch}"] = (g0, L, s0)
    s = s0.clone()
    s[0, 3] = v
    cases["scene"] = (g0, L0, s)
    with GlassNet(wts, W, k_max=K, precision="fp32") as net:
        for what, (g, L, s) in cases.items():
            ref = glassnet64(flat, *columns(g, L, s), fmax0).t().reshape(1, 3, H, WD)
            compare(net.forward(g, L, s), ref, f"W={W} {value}, {what}")
            st = net.stream_state(1, H, WD, device="cuda:0")
            net.stream_begin(g, s, st)
            for i in range(K):
                net.stream_accumulate(L[:, i:i + 1].contiguous(), st)
            compare(net.stream_finish(g, st), ref, f"W={W} {value}, {what}, streamed")
            net.stream_release(st)


@pytest.mark.parametrize("W", [64, 128])
@pytest.mark.parametrize("value", ["inf", "-inf"])
def test_fp32_forward_with_an_infinite_weight(W, value):
    wts, g, L, s = frame(W)
    wts[100] = VALUES[value]                         # F's first layer, row 3
    ref = glassnet64(layers_of(wts, synth.layer_shapes(W)), *columns(g, L, s), fmax0)
    with GlassNet(wts, W, k_max=K, precision="fp32") as net:
        compare(net.forward(g, L, s), ref.t().reshape(1, 3, H, WD), f"W={W} {value} weight")


@pytest.mark.parametrize("W", [64, 128])
def test_fp32_forward_of_the_largest_finite_value(W):
    """3.4e38 (bf16 ends at 3.39e38) by way of one neuron a layer."""
    torch = torch_dev()
    wts = np.zeros(synth.num_params(W), np.float32)
    for m in layers_of(wts, synth.layer_shapes(W)):
        assert not m.any()
    at = {}
    off = 0
    for i, (o, n) in enumerate(synth.layer_shapes(W)):
        at[i] = off, n
        off += o * n + o
    for i, col, x in ((9, W, 1.0), (10, 0, 0.75), (11, 0, 2.0 ** -100)):
        wts[at[i][0] + col] = x                      # row 0
    _, g, L, s = frame(W)
    g[0, 11] = 3.4e38
    with GlassNet(wts, W, k_max=K, precision="fp32") as net:
        y = net.forward(g, L, s)
    want = float(np.float32(3.4e38)) * 0.75 * 2.0 ** -100
    assert torch.all((y[0, 0].double() / want - 1).abs() <= 1e-6)
    assert not y[0, 1:].any()


@pytest.mark.parametrize("W", [64, 128])
@pytest.mark.parametrize("value", list(VALUES))
def test_backward_of_an_infinite_loss_gradient(W, value):
    """Which entries of the gradient are finite, and their values."""
    torch = torch_dev()
    wts, g, L, s = frame(W)
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    dy = torch.randn((1, 3, H, WD), generator=gen, device="cuda:0")
    dy[0, 1, 6, 9] = VALUES[value]
    flat = layers_of(wts, synth.layer_shapes(W))
    margins = []

    def relu(z):
        margins.append(z.detach().abs().amin(1))
        return torch.relu(z)
    y = glassnet64(flat, *columns(g, L, s), relu)
    dy *= (torch.stack(margins).amin(0) > 1e-5).float().reshape(H, WD)
    ref = torch.cat([t.reshape(-1) for t in torch.autograd.grad(
        y, flat, dy[0].double().reshape(3, -1).t())])
    assert not bool(torch.isfinite(ref).all()) and bool(torch.isfinite(ref).any())
    with GlassNet(wts, W, k_max=K, precision="fp32") as net:
        out = net.backward(g, L, s, dy).double()
    m = torch.isfinite(ref)
    assert torch.equal(torch.isfinite(out), m)
    last = ref.numel() - 3 * W - 3                   # R's last layer: one product each
    inf = torch.isinf(ref[last:])
    assert torch.equal(out[last:][inf], ref[last:][inf])
    err = float((out[m] - ref[m]).norm() / ref[m].norm())
    log(f"  W={W} {value}: {int((~m).sum())} of {m.numel()} not finite, others relF {err:.1e}")
    assert err <= 1e-5


@pytest.mark.parametrize("W", [64, 128])
@pytest.mark.parametrize("h,w", [(2, 5), (24, 40)])
def test_backward_of_the_largest_finite_deltas(W, h, w):
    """dL/dy of one pixel, R's last layer +-1, scaled by the power of two that takes
    the gradient's largest entry just below 2^128: with deltas from 2^126 on (a
    bias's gradient is that pixel's delta) the weight gradients take the split
    with clamps.  Every rounding commutes with the factor: all bits are the same."""
    torch = torch_dev()
    wts, g, L, s = frame(W)
    # (small inputs: no entry is much larger than the deltas)
    g, L, s = (0.25 * t for t in (g[..., :h, :w], L[..., :h, :w], s))
    last = wts.size - 3 * W - 3
    wts[last:-3] = np.sign(wts[last:-3])
    dy = torch.zeros((1, 3, h, w), device="cuda:0")
    dy[0, 1, 1, 3] = 1.0
    with GlassNet(wts, W, k_max=K, precision="fp32") as net:
        one = net.backward(g, L, s, dy)
        factor = 2.0 ** int(127.9 - np.log2(float(one.abs().max())))
        out = net.backward(g, L, s, dy * factor)
    at, deltas = 0, []
    for o, i in synth.layer_shapes(W):
        deltas.append(float(out[at + o * i:at + o * i + o].abs().max()))
        at += o * i + o
    assert sum(d >= 2.0 ** 126 for d in deltas) >= 1
    assert int((one != 0).sum()) > one.numel() // 8
    assert bool(torch.isfinite(out).all())
    assert torch.equal(out, one * factor)


def sr_inputs(n=1, h=20, w=24):
    torch = torch_dev()
    gen = torch.Generator(device="cuda:0").manual_seed(2)
    r = lambda *s: torch.rand(s, generator=gen, device="cuda:0") * 2 - 1  # noqa: E731
    return (synth.make_sr_weights(np.random.default_rng(3)), r(n, 3, h, w), r(n, 14, 2 * h, 2 * w),
            r(n, 3, 2 * h, 2 * w))


def sr64(flat, lo, g, relu):
    torch = torch_dev()
    up = lo.double()
    for d in (2, 3):
        m = up.shape[d]
        i = torch.arange(m, device=up.device)
        a, b = up.index_select(d, (i - 1).clamp_min(0)), up.index_select(d, (i + 1).clamp_max(m - 1))
        up = torch.stack([0.25 * a + 0.75 * up, 0.75 * up + 0.25 * b], d + 1).flatten(d, d + 1)
    x = torch.cat([up, g.double()], 1)[0].permute(1, 2, 0)
    a1 = relu(conv64(x, flat[0], flat[1], 3))
    return up + conv64(relu(conv64(a1, flat[2], flat[3], 3)), flat[4], flat[5], 1).permute(2, 0, 1)[None]


@pytest.mark.parametrize("value", list(VALUES))
def test_sr_forward(value):
    wts, lo0, g0, _ = sr_inputs()
    flat = layers_of(wts, SR_SHAPES)
    with GlassNet(None, 64, precision="fp32") as net:
        w = torch_dev().from_numpy(wts).to("cuda:0")
        for what, (c, y, x) in {"G-buffer": (3, 17, 21), "last channel": (13, 15, 16)}.items():
            g = g0.clone()
            g[0, c, y, x] = VALUES[value]
            compare(net.sr_forward(w, lo0, g), sr64(flat, lo0, g, fmax0), f"{value}, {what}")
        lo = lo0.clone()
        lo[0, 1, 9, 11] = VALUES[value]
        compare(net.sr_forward(w, lo, g0), sr64(flat, lo, g0, fmax0), f"{value}, render")


@pytest.mark.parametrize("value", list(VALUES))
def test_sr_backward(value):
    torch = torch_dev()
    wts, lo, g, dy = sr_inputs()
    dy[0, 1, 17, 21] = VALUES[value]
    flat = layers_of(wts, SR_SHAPES)
    ref = torch.cat([t.reshape(-1) for t in torch.autograd.grad(sr64(flat, lo, g, torch.relu), flat,
                                                                dy.double())])
    with GlassNet(None, 64, precision="fp32") as net:
        out = net.sr_backward(torch.from_numpy(wts).to("cuda:0"), lo, g, dy).double()
    m = torch.isfinite(ref)
    assert torch.equal(torch.isfinite(out), m)
    for a, b in zip(out.split([32 * 17 * 9, 32, 32 * 32 * 9, 32, 96, 3]),
                    ref.split([32 * 17 * 9, 32, 32 * 32 * 9, 32, 96, 3])):
        f = torch.isfinite(b)
        if bool(f.any()):                            # (a kink taken the other way: 1e-4, as elsewhere)
            assert float((a[f] - b[f]).norm()) <= 1e-4 * float(b[f].norm())
