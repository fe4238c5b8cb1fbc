"""GPU parity of object streaming through the C ABI: begin / accumulate /
finish over a frame whose transparent objects arrive a few at a time
(Sec. 3.3, Eq. (5): tau is a sum over transparency buffers; Sec. 4.4.2: each
object's buffer is evaluated on its own and added to a running sum).

The state keeps the running sum in fp32 and the library adds the slots in
call order, exactly as the fused forward of a handle with the input slot
order adds them in slot order, so a streamed result must equal that fused
forward over the concatenated slots bit for bit (GN_FP32 handles stream
through the plane pipeline of their forward, with the same property).  Against the FP64 oracle
the tolerances are the forward's (relative Frobenius error: fp32 1e-4, bf16
2e-2, fp8_t 6e-2).
"""
import numpy as np
import pytest

import oracle
from paper_2405_19056_amd import synth
from paper_2405_19056_amd.glassnet import GlassNet, GlassNetError, GN_E_INVAL

from gpu_util import dev, host, log, relF, torch_dev

pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-4, "bf16": 2e-2, "fp8_t": 6e-2}


def frame(n, h, w, k, W, seed):
    s = synth.streams(seed)
    wts = synth.make_weights(W, s["weights"])
    fr = synth.Frame(synth.make_gbuf(n, h, w, s["gbuf"]),
                     synth.make_layers(n, k, h, w, s["slots"], s["active"], "uniform_count"),
                     synth.make_scene(n, s["gbuf"]))
    return wts, fr


def open_net(wts, W, precision, pool="mean", k_max=8, slot_order="input"):
    net = GlassNet(wts, W, k_max=k_max, pool=pool, precision=precision, slot_order=slot_order)
    if precision == "fp8_t":
        _, cal = frame(1, 64, 64, 4, W, seed=999)
        net.calibrate(dev(cal.gbuf), dev(cal.layers), dev(cal.scene))
    return net


def fused(net, fr, k=None):
    torch = torch_dev()
    k = fr.k if k is None else k
    L = dev(fr.layers[:, :k]) if k > 0 else None
    y = net.forward(dev(fr.gbuf), L, dev(fr.scene))
    torch.cuda.synchronize()
    return host(y)


def streamed(net, fr, chunks, order=None, progressive=False):
    """Stream fr's slots in batches of the given sizes (slot order `order`)."""
    torch = torch_dev()
    order = list(range(fr.k)) if order is None else list(order)
    assert sum(chunks) == len(order)
    g, s = dev(fr.gbuf), dev(fr.scene)
    st = net.stream_state(fr.n, fr.h, fr.w)
    net.stream_begin(g, s, st)
    outs, i = [], 0
    for c in chunks:
        net.stream_accumulate(dev(fr.layers[:, order[i:i + c]]), st)
        i += c
        if progressive:
            outs.append(host(net.stream_finish(g, st)))
    y = net.stream_finish(g, st)
    torch.cuda.synchronize()
    net.stream_release(st)
    return host(y), outs


@pytest.mark.parametrize("precision,W,pool", [("bf16", 128, "mean"), ("bf16", 64, "sum"),
                                              ("fp8_t", 128, "mean"), ("fp8_t", 128, "sum"),
                                              ("fp32", 128, "mean"), ("fp32", 64, "sum")])
def test_streamed_frame_is_the_fused_forward_bitwise(precision, W, pool):
    wts, fr = frame(2, 37, 41, 5, W, seed=71)
    log(f"stream {precision} W={W} {pool} 2x37x41 K=5 chunks 2,0,1,2")
    with open_net(wts, W, precision, pool) as net:
        y_ref = fused(net, fr)
        y, _ = streamed(net, fr, [2, 0, 1, 2])
    assert np.array_equal(y, y_ref)
    e = relF(y, oracle.forward(wts, W, fr.gbuf, fr.layers, fr.scene, pool=pool))
    log(f"  relF vs oracle {e:.3e}")
    assert e <= TOL[precision]


@pytest.mark.parametrize("precision", ["bf16", "fp32"])
def test_progressive_results_after_each_object(precision):
    wts, fr = frame(1, 50, 61, 4, 128, seed=72)
    with open_net(wts, 128, precision) as net:
        _, outs = streamed(net, fr, [1, 1, 1, 1], progressive=True)
        for i, y in enumerate(outs):
            assert np.array_equal(y, fused(net, fr, k=i + 1)), i


@pytest.mark.parametrize("precision,W,first", [("bf16", 128, 0), ("bf16", 64, 1), ("fp8_t", 128, 2),
                                               ("fp32", 64, 0), ("fp32", 128, 1)])
def test_objects_covering_parts_of_the_frame_leave_the_rest(precision, W, first):
    """Slot 0 covers nothing, slot 1 every third pixel, slot 2 a rectangle;
    state memory that held NaN: pixels without objects are an empty pool."""
    torch = torch_dev()
    log(f"stream parts {precision} W={W} first={first}")
    wts, fr = frame(1, 23, 45, 3, W, seed=41)
    alpha = np.zeros((3, 23, 45), np.float32)
    alpha[1].reshape(-1)[::3] = 0.5
    alpha[2, 4:19, 7:40] = 0.25
    fr.layers[0, :, 9] = alpha
    order = [(first + i) % 3 for i in range(3)]
    with open_net(wts, W, precision) as net:
        sub = synth.Frame(fr.gbuf, np.ascontiguousarray(fr.layers[:, order]), fr.scene)
        want = fused(net, sub)
        g, sc = dev(fr.gbuf), dev(fr.scene)
        st = net.stream_state(1, 23, 45)
        st[: st.numel() // 4 * 4].view(torch.float32).fill_(float("nan"))
        net.stream_begin(g, sc, st)
        for i in order:
            net.stream_accumulate(dev(fr.layers[:, i:i + 1]), st)
        y = host(net.stream_finish(g, st))
        net.stream_release(st)
    np.testing.assert_array_equal(y, want)


@pytest.mark.parametrize("precision", ["bf16", "fp32"])
def test_no_objects_is_the_k0_forward(precision):
    wts, fr = frame(2, 23, 29, 3, 128, seed=73)
    with open_net(wts, 128, precision) as net:
        y, _ = streamed(net, fr, [], order=[])
        assert np.array_equal(y, fused(net, fr, k=0))
    ref = oracle.forward(wts, 128, fr.gbuf, np.zeros((2, 0, 12, 23, 29)), fr.scene, pool="mean")
    assert relF(y, ref) <= TOL[precision]


def test_object_order_does_not_matter():
    """Eq. (5) is symmetric in the objects: a permuted arrival order agrees with
    the oracle, and with the in-order stream up to fp32 summation order."""
    wts, fr = frame(1, 40, 44, 6, 128, seed=74)
    ref = oracle.forward(wts, 128, fr.gbuf, fr.layers, fr.scene, pool="mean")
    with open_net(wts, 128, "bf16") as net:
        y0, _ = streamed(net, fr, [3, 3])
        y1, _ = streamed(net, fr, [1, 2, 3], order=[5, 2, 0, 4, 1, 3])
    assert relF(y1, ref) <= TOL["bf16"]
    assert relF(y1, y0) <= 2e-3


def test_two_states_interleaved_on_one_handle():
    torch = torch_dev()
    wts, fa = frame(1, 33, 35, 4, 128, seed=75)
    _, fb = frame(2, 17, 70, 3, 128, seed=76)
    with open_net(wts, 128, "bf16") as net:
        ya, yb = fused(net, fa), fused(net, fb)
        sa, sb = net.stream_state(1, 33, 35), net.stream_state(2, 17, 70)
        net.stream_begin(dev(fa.gbuf), dev(fa.scene), sa)
        net.stream_begin(dev(fb.gbuf), dev(fb.scene), sb)
        net.stream_accumulate(dev(fa.layers[:, :2]), sa)
        net.stream_accumulate(dev(fb.layers[:, :1]), sb)
        net.stream_accumulate(dev(fa.layers[:, 2:]), sa)
        net.stream_accumulate(dev(fb.layers[:, 1:]), sb)
        oa = host(net.stream_finish(dev(fa.gbuf), sa))
        ob = host(net.stream_finish(dev(fb.gbuf), sb))
        torch.cuda.synchronize()
    assert np.array_equal(oa, ya) and np.array_equal(ob, yb)


def test_rebegun_state_starts_from_an_empty_pool():
    torch = torch_dev()
    wts, fa = frame(1, 30, 30, 3, 128, seed=77)
    _, fb = frame(1, 30, 30, 2, 128, seed=78)
    with open_net(wts, 128, "bf16") as net:
        st = net.stream_state(1, 30, 30)
        net.stream_begin(dev(fa.gbuf), dev(fa.scene), st)
        net.stream_accumulate(dev(fa.layers), st)
        net.stream_begin(dev(fb.gbuf), dev(fb.scene), st)
        net.stream_accumulate(dev(fb.layers), st)
        y = host(net.stream_finish(dev(fb.gbuf), st))
        torch.cuda.synchronize()
        assert np.array_equal(y, fused(net, fb))


def test_stream_argument_errors():
    torch = torch_dev()
    wts, fr = frame(1, 20, 24, 2, 128, seed=79)
    g, s, L = dev(fr.gbuf), dev(fr.scene), dev(fr.layers)
    with open_net(wts, 128, "bf16", k_max=2) as net:
        st = net.stream_state(1, 20, 24)
        with pytest.raises(GlassNetError) as e:       # never begun
            net.stream_accumulate(L, st)
        assert e.value.status == GN_E_INVAL
        with pytest.raises(GlassNetError) as e:       # too small for the frame
            net.stream_begin(g, s, st[: st.numel() // 2])
        assert e.value.status == GN_E_INVAL
        net.stream_begin(g, s, st)
        with pytest.raises(GlassNetError) as e:       # geometry differs from begin
            net.stream_accumulate(dev(fr.layers[:, :, :, :10]), st)
        assert e.value.status == GN_E_INVAL
        with pytest.raises(GlassNetError) as e:       # k above k_max
            net.stream_accumulate(torch.cat([L, L], dim=1), st)
        assert e.value.status == GN_E_INVAL
        with pytest.raises(GlassNetError) as e:       # out aliases the state
            net.stream_finish(g, st, out=st[: 3 * 20 * 24 * 4].view(torch.float32).view(1, 3, 20, 24))
        assert e.value.status == GN_E_INVAL
        net.stream_release(st)
        with pytest.raises(GlassNetError) as e:       # released
            net.stream_finish(g, st)
        assert e.value.status == GN_E_INVAL


def test_state_size_does_not_grow_with_objects():
    wts, _ = frame(1, 8, 8, 1, 128, seed=80)
    with GlassNet(wts, 128, k_max=64, precision="bf16") as net:
        b = net.stream_state_bytes(1, 512, 512)
        assert b == 512 * 512 * 772
        with GlassNet(synth.make_weights(64, np.random.default_rng(0)), 64,
                      precision="bf16") as n64:
            assert n64.stream_state_bytes(3, 7, 100) == 3 * 3 * 256 * 388
    with GlassNet(wts, 128, k_max=64, precision="fp32") as net:
        assert net.stream_state_bytes(2, 30, 50) == 2 * 30 * 50 * (2 * 128 + 1) * 4


@pytest.mark.parametrize("precision", ["bf16", "fp8_t", "fp32"])
def test_full_512sq_k8_one_object_per_call(precision):
    """The 512^2, K=8, W=128 workload streamed one object per call."""
    w, fr, _ = synth.config_inputs("c2_512sq_k8_w128")
    log(f"stream 512^2 K=8 {precision}, one object per call")
    with open_net(w, 128, precision) as net:
        y_ref = fused(net, fr)
        y, _ = streamed(net, fr, [1] * 8)
    assert np.array_equal(y, y_ref)


@pytest.mark.parametrize("precision,W", [("bf16", 128), ("bf16", 64), ("fp8_t", 128)])
@pytest.mark.parametrize("h,w_", [(192, 192), (193, 192), (262, 271)])
def test_partly_covered_frames_of_few_and_many_tiles(precision, W, h, w_):
    """144 tiles (nine for 16 of 256 CUs: the state kept 16 pixels at a time), 145,
    and 278 (some workgroups take two); state memory that held NaN, objects that
    cover nothing, stripes and a rectangle, a result after every call."""
    torch = torch_dev()
    log(f"stream {precision} W={W} {h}x{w_} in parts")
    wts, fr = frame(1, h, w_, 4, W, seed=h)
    alpha = np.zeros((4, h, w_), np.float32)
    alpha[1].reshape(-1)[::3] = 0.5
    alpha[2, h // 4:h - 40, 30:w_ - 50] = 0.25
    alpha[3, :, : w_ // 2] = 1.0
    fr.layers[0, :, 9] = alpha
    with open_net(wts, W, precision) as net:
        g, sc = dev(fr.gbuf), dev(fr.scene)
        st = net.stream_state(1, h, w_)
        st[: st.numel() // 4 * 4].view(torch.float32).fill_(float("nan"))
        net.stream_begin(g, sc, st)
        np.testing.assert_array_equal(host(net.stream_finish(g, st)), fused(net, fr, k=0))
        for first, last in ((0, 1), (1, 2), (2, 4)):
            net.stream_accumulate(dev(fr.layers[:, first:last]), st)
            np.testing.assert_array_equal(host(net.stream_finish(g, st)), fused(net, fr, k=last))
        net.stream_release(st)
