"""Super-sampling of frames whose G-buffer takes more than 2 GiB, 4 GiB, and
whose single planes take more than 2 GiB: parts of the output equal, bitwise,
those of the same parts super-sampled on their own (an output depends on the
input within three pixels of it)."""
import numpy as np
import pytest

from paper_2405_19056_amd import synth
from paper_2405_19056_amd.glassnet import GlassNet

from gpu_util import log, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w", [(4096, 4096), (5121, 4099), (64, 1 << 18), (16384, 8200)])
def test_large_frames(h, w):
    torch = torch_dev()
    log(f"  super-sampling {h}x{w}: {14 * 16 * h * w / 2**30:.1f} GiB of G-buffer")
    gen = torch.Generator(device="cuda:0").manual_seed(h)
    lo = torch.rand((1, 3, h, w), generator=gen, device="cuda:0")
    g = torch.empty((1, 14, 2 * h, 2 * w), device="cuda:0")
    for c in range(14):
        torch.rand(g[0, c].shape, generator=gen, device="cuda:0", out=g[0, c])
    wts = torch.from_numpy(synth.make_sr_weights(np.random.default_rng(1))).to("cuda:0")
    with GlassNet(None, 64, precision="fp32") as net:
        y = net.sr_forward(wts, lo, g)
        ch, cw = 32, 40                      # a part's size; its corners in the frame
        for r in (0, (h - ch) // 16 * 8, h - ch):
            for c in (0, (w - cw) // 16 * 8, w - cw):
                part = net.sr_forward(wts, lo[:, :, r:r + ch, c:c + cw].contiguous(),
                                      g[:, :, 2 * r:2 * (r + ch), 2 * c:2 * (c + cw)].contiguous())
                # away from the part's edges, but for those that are the frame's
                t, b = (0 if r == 0 else 4), (2 * ch if r == h - ch else 2 * ch - 4)
                le, ri = (0 if c == 0 else 4), (2 * cw if c == w - cw else 2 * cw - 4)
                whole = y[:, :, 2 * r + t:2 * r + b, 2 * c + le:2 * c + ri]
                assert bool(whole.abs().sum() > 0)
                assert torch.equal(whole, part[:, :, t:b, le:ri]), (r, c)
    del g, y, lo
    torch.cuda.empty_cache()
