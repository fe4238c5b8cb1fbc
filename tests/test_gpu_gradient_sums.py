"""Rounding of the weight gradients' long sums, against a plain torch evaluation
in 64 bits.

The gradients' matrix products run on an instruction that rounds towards minus
infinity.  A rounding that goes either way grows with the square root of the
number of pixels, as a sum of random signs itself does; a one-sided one grows
with their number, and is 10^-5 of a gradient over 2^18 pixels.  So the sums are
checked where dL/dy is random and sits where a scheme of alternating signs could
not cancel it: in every second wave's pixels or tile, or in one block of a frame.

dL/dy is zero on pixels within 2e-5 of a ReLU's kink, which fp32 may evaluate on
the other side.
"""
import numpy as np
import pytest

from paper_2405_19056_amd import synth
from paper_2405_19056_amd.glassnet import GlassNet

from gpu_util import log, torch_dev
from ref64 import SR_SHAPES, columns, conv64, glassnet64, layers_of

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float((a - b).norm() / b.norm())


def glassnet_grad64(flat, G, L, S, dy):
    """Gradient of sum(dy y) over pixels, and dy, zeroed near kinks."""
    torch = torch_dev()
    margins = []

    def relu(z):
        margins.append(z.detach().abs().amin(1))
        return torch.relu(z)
    y = glassnet64(flat, G, L, S, relu)
    dy = dy * (torch.stack(margins).amin(0) > 2e-5)[:, None]
    return torch.cat([t.reshape(-1) for t in torch.autograd.grad((y * dy).sum(), flat)]), dy


WHERE = {
    "everywhere": lambda p: p >= 0,
    "every second wave": lambda p: (p // 16) % 2 == 0,
    "one block": lambda p: (p >= 65536) & (p < 65536 + 7680),
}


@pytest.mark.parametrize("W", [64, 128])
@pytest.mark.parametrize("where", list(WHERE))
def test_backward_sums_over_many_pixels(W, where):
    """2^18 pixels, K = 2.  Bar: a delta passes at most ten maps, whose fp32 sums
    are off by up to three units of 2^-24 each, independently from pixel to
    pixel: 10 x 3 x 2^-24 = 1.8e-6 of the gradient, whatever the count."""
    torch = torch_dev()
    h, w_, k = 256, 1024, 2
    wts = synth.make_weights(W, np.random.default_rng(5))
    gen = torch.Generator(device="cuda:0").manual_seed(11)
    g = torch.rand((1, 14, h, w_), generator=gen, device="cuda:0") * 2 - 1
    L = torch.rand((1, k, 12, h, w_), generator=gen, device="cuda:0") * 2 - 1
    s = torch.rand((1, 16), generator=gen, device="cuda:0") * 2 - 1
    dy = torch.randn((h * w_, 3), generator=gen, device="cuda:0").double()
    dy *= WHERE[where](torch.arange(h * w_, device="cuda:0"))[:, None]
    flat = layers_of(wts, synth.layer_shapes(W))
    G, Ls, S = columns(g, L, s)
    ref, ds, step = 0, [], 1 << 15
    for i in range(0, h * w_, step):
        gr, d = glassnet_grad64(flat, G[i:i + step], Ls[i:i + step], S[i:i + step], dy[i:i + step])
        ref = ref + gr
        ds.append(d)
    d = torch.cat(ds).float().t().reshape(1, 3, h, w_).contiguous()
    with GlassNet(wts, W, k_max=k, precision="fp32") as net:
        err = rel(net.backward(g, L, s, d).double(), ref)
    log(f"  backward W={W}, dL/dy {where}: relF {err:.2e}")
    assert err <= 1.8e-6


@pytest.mark.parametrize("where", ["every tile", "every second tile"])
def test_sr_gradient_sums_over_many_pixels(where):
    """8 frames of 64^2 -> 128^2 (2^17 pixels), conv1's gradient.  Bar: its
    deltas are fp32 sums over nine taps of 32 products, off by up to nine units
    of 2^-24, independently from pixel to pixel, and so are the sums over the
    pixels: 2 x 9 x 2^-24 = 1.1e-6."""
    torch = torch_dev()
    n, h, w_ = 8, 64, 64
    wts = synth.make_sr_weights(np.random.default_rng(6))
    gen = torch.Generator(device="cuda:0").manual_seed(12)
    # the render is constant, so that its upsampling has no rounding
    lo = torch.full((n, 3, h, w_), 0.5, device="cuda:0")
    g = torch.rand((n, 14, 2 * h, 2 * w_), generator=gen, device="cuda:0") * 2 - 1
    dy = torch.randn((n, 3, 2 * h, 2 * w_), generator=gen, device="cuda:0")
    tile = torch.arange(2 * h, device="cuda:0")[:, None] // 16 + torch.arange(2 * w_, device="cuda:0") // 16
    if where == "every second tile":
        dy *= tile % 2 == 0
    flat = layers_of(wts, SR_SHAPES)
    ref = 0
    for f in range(n):
        x = torch.cat([torch.full((2 * h, 2 * w_, 3), 0.5, device="cuda:0", dtype=torch.float64),
                       g[f].double().permute(1, 2, 0)], 2)
        z1 = conv64(x, flat[0], flat[1], 3)
        z2 = conv64(torch.relu(z1), flat[2], flat[3], 3)
        m = torch.minimum(z1.detach().abs().amin(2), z2.detach().abs().amin(2))
        near = torch.nn.functional.max_pool2d((m < 2e-6).double()[None, None], 3, 1, 1)[0, 0]
        dy[f] *= (near == 0).float()
        y = conv64(torch.relu(z2), flat[4], flat[5], 1)
        ref = ref + torch.cat([t.reshape(-1) for t in torch.autograd.grad(
            (y * dy[f].double().permute(1, 2, 0)).sum(), flat)])
    with GlassNet(None, 64, precision="fp32") as net:
        out = net.sr_backward(torch.from_numpy(wts).to("cuda:0"), lo, g, dy).double()
    m = 32 * 17 * 9
    err = max(rel(out[:m], ref[:m]), rel(out[m:m + 32], ref[m:m + 32]))
    log(f"  super-sampling gradient, dL/dy in {where}: conv1 relF {err:.2e}")
    assert err <= 1.1e-6
