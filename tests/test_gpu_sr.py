"""GPU x2 super-sampling network (glassnet_sr_forward; Sec. 3.4 doubles the
render's resolution with a small CNN fed by full-resolution G-buffers)
against the FP64 oracle, through the C ABI.

Bar: relF <= 1e-5 over every output (fp32 sums of at most 288 products per
conv output, then a 32-term head: a few fp32 ulps of the largest terms).
Shapes span several 16 x 16 output tiles with ragged edges, a single tile,
a 1 x 1 render (every tap but the centre in the zero padding) and the
256^2 -> 512^2 frame of the paper's pipeline, compared whole.
"""
import numpy as np
import pytest

import oracle
from paper_2405_19056_amd import synth
from paper_2405_19056_amd.glassnet import GlassNet, GlassNetError, GN_E_INVAL, lib

from gpu_util import dev, host, log, relF, torch_dev

pytestmark = pytest.mark.gpu


def net64():
    return GlassNet(synth.make_weights(64, np.random.default_rng(0)), 64, precision="bf16")


def run(net, w, lo, g):
    torch = torch_dev()
    y = net.sr_forward(dev(w), dev(lo), dev(g))
    torch.cuda.synchronize()
    return host(y)


@pytest.mark.parametrize("n,h,w", [(2, 19, 23), (1, 8, 8), (1, 1, 1), (1, 3, 17), (3, 9, 5),
                                   (64, 8, 8), (1, 2, 300)])
def test_sr_matches_oracle(n, h, w):
    wts = synth.make_sr_weights(np.random.default_rng(h * 100 + w))
    lo, g = synth.make_sr_inputs(n, h, w, seed=h * w + n)
    ref = oracle.sr_forward(wts, lo, g)
    with net64() as net:
        y = run(net, wts, lo, g)
    err = relF(y, ref)
    log(f"sr {n}x{h}x{w} -> {2 * h}x{2 * w}: relF {err:.2e}")
    assert y.shape == ref.shape
    assert err <= 1e-5


@pytest.mark.parametrize("n,h,w", [(1, 7, 9), (2, 8, 16), (1, 9, 7), (1, 17, 24), (1, 1, 8)])
def test_sr_forward_and_gradient_at_tile_edges(n, h, w):
    """Outputs of 14, 16, 18 and 34 rows or columns around the 16 x 16 tiles,
    every channel of the input on its own scale (the operands are split in
    three per value); the bars of the tests around this one."""
    torch = torch_dev()
    wts = synth.make_sr_weights(np.random.default_rng(h * 31 + w))
    lo, g = synth.make_sr_inputs(n, h, w, seed=3 * h + w)
    g = g * (10.0 ** np.arange(-6, 8)).astype(np.float32)[None, :, None, None] ** 0.25
    g = np.ascontiguousarray(g, dtype=np.float32)
    dy = np.random.default_rng(h + w).normal(size=(n, 3, 2 * h, 2 * w)).astype(np.float32)
    log(f"sr tile edges {n}x{h}x{w}")
    with net64() as net:
        y = run(net, wts, lo, g)
        gw = net.sr_backward(dev(wts), dev(lo), dev(g), dev(dy))
        torch.cuda.synchronize()
        gw = host(gw)
    assert relF(y, oracle.sr_forward(wts, lo, g)) <= 1e-5
    errs = _per_tensor_relF(gw, oracle.sr_grad(wts, lo, g, dy))
    assert max(errs.values()) <= 1e-4, errs


def test_sr_full_frame_256_to_512():
    wts = synth.make_sr_weights(np.random.default_rng(7))
    lo, g = synth.make_sr_inputs(1, 256, 256, seed=7)
    ref = oracle.sr_forward(wts, lo, g)
    with net64() as net:
        y = run(net, wts, lo, g)
    err = relF(y, ref)
    log(f"sr 256^2 -> 512^2: relF {err:.2e}, max |err| {np.max(np.abs(y - ref)):.2e}")
    assert err <= 1e-5


def test_zero_weights_give_upsample_plus_bias():
    wts = np.zeros(oracle.sr_n_params(), np.float32)
    wts[-3:] = (0.5, -1.0, 2.0)
    lo, g = synth.make_sr_inputs(1, 13, 10, seed=3)
    with net64() as net:
        y = run(net, wts, lo, g)
    want = oracle.upsample2x(lo) + np.array([0.5, -1.0, 2.0])[None, :, None, None]
    assert np.max(np.abs(y - want)) <= 1e-6


def test_consecutive_calls_pick_up_new_weights_and_sizes():
    w1 = synth.make_sr_weights(np.random.default_rng(11))
    w2 = synth.make_sr_weights(np.random.default_rng(12))
    lo1, g1 = synth.make_sr_inputs(2, 24, 20, seed=11)
    lo2, g2 = synth.make_sr_inputs(1, 7, 9, seed=12)
    with net64() as net:
        y1 = run(net, w1, lo1, g1)
        y2 = run(net, w2, lo2, g2)
    assert relF(y1, oracle.sr_forward(w1, lo1, g1)) <= 1e-5
    assert relF(y2, oracle.sr_forward(w2, lo2, g2)) <= 1e-5


def test_sr_argument_errors():
    torch = torch_dev()
    w = dev(synth.make_sr_weights(np.random.default_rng(0)))
    lo = torch.zeros((1, 3, 4, 4), device="cuda:0")
    g = torch.zeros((1, 14, 8, 8), device="cuda:0")
    out = torch.zeros((1, 3, 8, 8), device="cuda:0")
    with net64() as net:
        L = lib()
        for args in ((net._h, w.data_ptr(), 0, 4, 4, lo.data_ptr(), g.data_ptr(), out.data_ptr()),
                     (net._h, w.data_ptr(), 1, 0, 4, lo.data_ptr(), g.data_ptr(), out.data_ptr()),
                     (net._h, None, 1, 4, 4, lo.data_ptr(), g.data_ptr(), out.data_ptr()),
                     (net._h, w.data_ptr(), 1, 4, 4, lo.data_ptr(), g.data_ptr(), g.data_ptr()),
                     (net._h, w.data_ptr(), 1, 4, 4, lo.data_ptr(), g.data_ptr(),
                      lo.data_ptr() + 4)):
            assert L.glassnet_sr_forward(*args, None) == GN_E_INVAL
        with pytest.raises(ValueError):
            net.sr_forward(w, lo, torch.zeros((1, 14, 8, 9), device="cuda:0"))
        torch.cuda.synchronize()
        assert not out.any()                    # nothing ran


# ---------------------------------------------------------------- backward
def _per_tensor_relF(g, ref):
    out, o = {}, 0
    for name, shp in oracle.sr_oracle.sr_shapes():
        k = int(np.prod(shp))
        out[name] = relF(g[o:o + k], ref[o:o + k])
        o += k
    return out


@pytest.mark.parametrize("n,h,w", [(2, 19, 23), (1, 8, 8), (1, 1, 1), (16, 32, 32), (40, 4, 6),
                                   (1, 3, 200)])
def test_sr_backward_matches_oracle(n, h, w):
    """Against the FP64 oracle's gradient, every tensor within relF 1e-4 (fp32
    sums over up to 2^16 pixels per weight, per-workgroup partials added in
    fp32 in a fixed order);
    repeated calls are bitwise equal."""
    torch = torch_dev()
    wts = synth.make_sr_weights(np.random.default_rng(h * 7 + w))
    lo, g = synth.make_sr_inputs(n, h, w, seed=h + w + n)
    dy = np.random.default_rng(n * h * w).normal(size=(n, 3, 2 * h, 2 * w)).astype(np.float32)
    ref = oracle.sr_grad(wts, lo, g, dy)
    with net64() as net:
        args = (dev(wts), dev(lo), dev(g), dev(dy))
        g1 = net.sr_backward(*args)
        g2 = net.sr_backward(*args)
        torch.cuda.synchronize()
        g1, g2 = host(g1), host(g2)
    errs = _per_tensor_relF(g1, ref)
    log(f"sr backward {n}x{h}x{w}: " + ", ".join(f"{k} {v:.2e}" for k, v in errs.items()))
    assert np.array_equal(g1, g2)
    assert max(errs.values()) <= 1e-4, errs


def test_sr_backward_argument_errors():
    torch = torch_dev()
    w = dev(synth.make_sr_weights(np.random.default_rng(0)))
    lo = torch.zeros((1, 3, 4, 4), device="cuda:0")
    g = torch.zeros((1, 14, 8, 8), device="cuda:0")
    dy = torch.zeros((1, 3, 8, 8), device="cuda:0")
    gw = torch.full((oracle.sr_n_params(),), 7.0, device="cuda:0")
    with net64() as net:
        L = lib()
        for args in ((net._h, w.data_ptr(), 1, 4, 4, lo.data_ptr(), g.data_ptr(), dy.data_ptr(),
                      w.data_ptr()),                                 # grad_w aliases sr_w
                     (net._h, w.data_ptr(), 1, 4, 4, lo.data_ptr(), g.data_ptr(), dy.data_ptr(),
                      None),
                     (net._h, w.data_ptr(), 2, 1024, 1024, lo.data_ptr(), g.data_ptr(),
                      dy.data_ptr(), gw.data_ptr())):                # beyond 2^22 output pixels
            assert L.glassnet_sr_backward(*args, None) == GN_E_INVAL
        torch.cuda.synchronize()
        assert bool((gw == 7.0).all())          # nothing ran


# ---------------------------------------------------------------- training
def test_adam_update_matches_oracle():
    """glassnet_adam_update on a caller-owned vector: three steps against the
    oracle's Adam (hyperparameters as the fp32 values that cross the ABI)."""
    torch = torch_dev()
    n = oracle.sr_n_params()
    rng = np.random.default_rng(41)
    f32 = lambda x: float(np.float32(x))  # noqa: E731
    lr, b1, b2, eps, wd = f32(1e-3), f32(0.9), f32(0.999), f32(1e-8), f32(1e-4)
    w0 = synth.make_sr_weights(rng)
    w, m, v = w0.astype(np.float64), np.zeros(n), np.zeros(n)
    with net64() as net:
        wd_dev, state = dev(w0), torch.zeros(2 * n, device="cuda:0")
        for t in range(1, 4):
            g = (rng.normal(size=n) * 10.0 ** rng.uniform(-4, 0, size=n)).astype(np.float32)
            net.adam_update(wd_dev, dev(g), state, t, lr=lr, betas=(b1, b2), eps=eps,
                            weight_decay=wd)
            w, m, v = oracle.adam_step(w, g, m, v, t, lr=lr, beta1=b1, beta2=b2, eps=eps,
                                       weight_decay=wd)
        torch.cuda.synchronize()
        assert float(np.max(np.abs(host(wd_dev) - w))) <= 1e-6
        st = host(state)
        assert relF(st[:n], m) <= 1e-5 and relF(st[n:], v) <= 1e-5
        with pytest.raises(GlassNetError) as e:                 # gradient inside the state
            net.adam_update(wd_dev, state[:n], state, 1)
        assert e.value.status == GN_E_INVAL


def test_sr_train_step():
    """One step of autograd.train_step_sr (L1 + DSSIM, weight gradient, Adam):
    both loss terms and the gradient against the oracle at the same weights,
    and the weights moved by exactly the Adam step of that gradient."""
    from paper_2405_19056_amd.autograd import train_step_sr
    torch = torch_dev()
    n, h, w = 2, 16, 20
    w0 = synth.make_sr_weights(np.random.default_rng(51))
    lo, g = synth.make_sr_inputs(n, h, w, seed=51)
    y_ref = oracle.sr_forward(w0, lo, g)
    tgt = (y_ref + 0.05 * np.random.default_rng(52).normal(size=y_ref.shape)).astype(np.float32)
    l1, dl1 = oracle.l1_loss(y_ref, tgt)
    ds, dds = oracle.dssim_loss(y_ref, tgt)
    gref = oracle.sr_grad(w0, lo, g, dl1 + dds)
    lr = float(np.float32(1e-3))
    with net64() as net:
        srw = dev(w0)
        state = torch.zeros(2 * w0.size, device="cuda:0")
        losses, gw = train_step_sr(net, srw, state, dev(lo), dev(g), dev(tgt), 1, lr=lr)
        torch.cuda.synchronize()
        losses, gw, w1 = host(losses), host(gw), host(srw)
    log(f"sr train step: L1 {losses[0]:.6f} vs {l1:.6f}, DSSIM {losses[1]:.6f} vs {ds:.6f}, "
        f"grad relF {relF(gw, gref):.2e}")
    assert abs(losses[0] - l1) <= 1e-6 * max(1.0, abs(l1))
    assert abs(losses[1] - ds) <= 2e-6
    assert relF(gw, gref) <= 1e-4
    want, _, _ = oracle.adam_step(w0.astype(np.float64), gw, np.zeros(w0.size), np.zeros(w0.size),
                                  1, lr=lr)
    assert float(np.max(np.abs(w1 - want))) <= 1e-6


def test_sr_backward_max_size_patch():
    """At the limit of 2^22 output pixels (4 renders of 512^2 -> 1024^2), with
    dL/d(out) non-zero on one 16 x 16 patch only: the weight gradient depends
    on the inputs within a few pixels of the patch, so the oracle's gradient on
    a 48 x 48 crop around it (crop edges 16 pixels from the patch, even-aligned
    for the upsample) is the exact answer; the call is also deterministic."""
    torch = torch_dev()
    n, h, w = 4, 512, 512
    wts = synth.make_sr_weights(np.random.default_rng(61))
    lo, g = synth.make_sr_inputs(n, h, w, seed=61)
    dy = np.zeros((n, 3, 2 * h, 2 * w), np.float32)
    dy[2, :, 496:512, 736:752] = np.random.default_rng(62).normal(size=(3, 16, 16))
    ref = oracle.sr_grad(wts, lo[2:3, :, 240:264, 360:384], g[2:3, :, 480:528, 720:768],
                         dy[2:3, :, 480:528, 720:768])
    with net64() as net:
        args = (dev(wts), dev(lo), dev(g), dev(dy))
        g1 = net.sr_backward(*args)
        g2 = net.sr_backward(*args)
        torch.cuda.synchronize()
        g1, g2 = host(g1), host(g2)
    errs = _per_tensor_relF(g1, ref)
    log("sr backward 4x512^2 patch: " + ", ".join(f"{k} {v:.2e}" for k, v in errs.items()))
    assert np.array_equal(g1, g2)
    assert max(errs.values()) <= 1e-4, errs


def test_sr_large_frame_sampled_crops():
    """A 1024 x 576 render (the largest serving frame) to 2048 x 1152: the
    oracle on 40 x 40 output crops at the corners and inside the frame; each
    output depends on inputs within 3 pixels, so the crop's inner part away
    from its cut edges is exact (image edges are real edges)."""
    wts = synth.make_sr_weights(np.random.default_rng(71))
    lo, g = synth.make_sr_inputs(1, 576, 1024, seed=71)
    with net64() as net:
        y = run(net, wts, lo, g)
    H, W = 1152, 2048
    for (Y0, X0) in ((0, 0), (H - 40, W - 40), (0, W - 40), (H - 40, 0), (560, 1000), (336, 1608)):
        ref = oracle.sr_forward(wts, lo[:, :, Y0 // 2:(Y0 + 40) // 2, X0 // 2:(X0 + 40) // 2],
                                g[:, :, Y0:Y0 + 40, X0:X0 + 40])
        # keep 6 pixels from every cut edge (not from the image's own edges)
        r0 = 0 if Y0 == 0 else 6
        r1 = 40 if Y0 + 40 == H else 34
        c0 = 0 if X0 == 0 else 6
        c1 = 40 if X0 + 40 == W else 34
        got = y[:, :, Y0 + r0:Y0 + r1, X0 + c0:X0 + c1]
        assert relF(got, ref[:, :, r0:r1, c0:c1]) <= 1e-5, (Y0, X0)
