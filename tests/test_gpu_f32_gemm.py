"""The fp32 implicit GEMM at the edges of its tiles, loads and splits: ragged
rows and columns of every tile, channel counts with and without whole
vectors, reductions of whole steps in one tap and not, more taps than a
tap mask holds, split and unsplit, strided phases with and without taps.

Bar: with accumulators that run over at most 256 products (the few-channel weight
gradient's over at most K / 4096, if that is more) and are then added up, every
result is within (256 + K / 256 + 40) * 2^-24 of the sum of its products'
magnitudes (K products; 40 bounds the split sums, the bias and the final
rounding), which the oracle gives from the magnitudes of the operands.
Random operands stay far below it whatever the chains; equal products, of a size
that the running sum rounds the same way each time, do not."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import paper_2404_12406_amd as ms
import synth
from paper_2404_12406_amd import _lib

from _gpu import dev, guarded_empty, guards_intact, host

pytestmark = pytest.mark.gpu


def _bar(k, magnitude):
    return (256 + k / 256 + 40) * 2.0 ** -24 * magnitude


def _within(name, got, ref, magnitude, k):
    bad = np.abs(got - ref) - _bar(k, magnitude)
    assert np.isfinite(got).all() and bad.max() <= 0, (name, float(np.abs(got - ref).max()), float(bad.max()))


CONVS = [
    # x shape, w shape, stride, pad
    ((4225, 64), (1030, 64), None, None),                    # 128 x 128 tiles, ragged both ways, tap steps
    ((4225, 66), (1030, 66), None, None),                    # the same size on 4-byte loads
    ((70, 36), (9, 36), None, None),                         # vectors, but no whole step
    ((33, 1), (1, 1), None, None),                           # one product, one column
    ((2, 32, 17, 19), (33, 32, 3, 3), (1, 1), (1, 1)),       # forward by tap steps, gradients on 4-byte loads
    ((2, 64, 15, 14), (96, 64, 3, 3), (2, 2), (1, 1)),       # strided: four phases by tap steps
    ((2, 32, 9, 10), (32, 32, 1, 1), (2, 2), (0, 0)),        # phases that no tap reaches
    ((1, 32, 6, 5), (32, 32, 6, 6), (1, 1), (3, 3)),         # 36 taps: more than a tap mask holds
    ((1, 64, 1, 1), (32, 64, 3, 3), (1, 1), (1, 1)),         # every tap but one in the padding
    ((1, 128, 4, 4), (256, 128, 3, 3), (1, 1), (1, 1)),      # a deep reduction of few tiles: split
    ((9, 8, 40, 37), (8, 8, 3, 3), (1, 1), (1, 1)),          # few channels both ways
    ((3, 20, 13, 11), (36, 20, 3, 2), (3, 2), (0, 1)),       # vectors across taps, uneven strides
    ((2, 5, 12, 12), (7, 5, 5, 5), (2, 1), (2, 1)),          # odd channels
    ((2, 3, 33, 30), (64, 3, 7, 7), (2, 2), (3, 3)),         # a stem
    # few channels and pixels enough for the kernels of their own
    ((9, 8, 101, 301), (8, 8, 3, 3), (1, 1), (1, 1)),        # every pass, ragged strips of rows and columns
    ((5, 3, 211, 251), (5, 3, 3, 3), (1, 1), (1, 0)),        # three input channels; five filters
    ((5, 4, 215, 251), (13, 4, 3, 2), (1, 2), (0, 1)),       # a column step of two, an even filter
    ((5, 16, 131, 403), (16, 16, 3, 3), (1, 1), (2, 2)),     # sixteen both ways, wide padding
    ((3, 1, 301, 301), (2, 1, 5, 5), (1, 1), (2, 2)),        # one channel, 5 x 5
    ((16, 4, 257, 259), (24, 4, 7, 7), (2, 2), (3, 3)),      # strided phases of the input gradient
    # few channels of one-pixel or small images: the GEMM's
    ((16500, 36), (1, 36), None, None),
    ((16500, 768), (10, 768), None, None),
    ((20001, 12), (16, 12), None, None),
    ((17000, 4, 1, 1), (5, 4, 3, 3), (1, 1), (1, 1)),
    ((420, 16, 13, 13), (16, 16, 3, 3), (1, 1), (1, 1)),
    ((33, 64, 56, 56), (4, 64, 1, 1), (1, 1), (0, 0)),
]


CHAINS = [
    # result, images, channels, extent, filters, filter extent, stride
    ("y", 16, 256, 64, 4, 3, 1),     # few channels out: chunks of four, 2304 products
    ("y", 16, 64, 64, 4, 5, 1),      # 1600, any number of filter rows
    ("y", 4, 3, 256, 2, 15, 1),      # 675, three channels at once
    ("dx", 4, 3, 224, 64, 7, 2),     # 1024, the stride phases of an input gradient
    ("y", 2, 256, 14, 64, 3, 1),     # the GEMM
    ("dx", 2, 64, 14, 256, 3, 1),
]


@pytest.mark.parametrize("case", range(len(CONVS)))
def test_f32_contractions(case):
    xs, ws, stride, pad = CONVS[case]
    seed = 9000 + 10 * case
    fan = int(np.prod(ws[1:]))
    x = synth.normal(xs, seed, dtype="f32")
    w = synth.kaiming_uniform(ws, seed + 1, fan, dtype="f32")
    b = synth.normal((ws[0],), seed + 2, 1.0, dtype="f32")
    if stride is None:
        spec = ms.Linear()
        f, dx, dw = oracle.linear_forward, lambda g, w: oracle.linear_input_grad(g, w), lambda g, x: oracle.linear_weight_grad(g, x)
    else:
        spec = ms.Conv2d(stride, pad)
        f = lambda x, w, b: oracle.conv2d_forward(x, w, b, stride, pad)
        dx = lambda g, w: oracle.conv2d_input_grad(g, w, xs, stride, pad)
        dw = lambda g, x: oracle.conv2d_weight_grad(g, x, ws, stride, pad)
    ref = f(x, w, b)
    gy = synth.normal(ref.shape, seed + 3, dtype="f32")
    X, W, B, G = (dev(t, "f32") for t in (x, w, b, gy))
    bufs = [guarded_empty(s, "f32") for s in (ref.shape, xs, ws, (ws[0],))]
    y, rec = ms.layer_forward(spec, X, W, B, 7, y=bufs[0][0])
    gx, gw, gb = ms.layer_backward(rec, G, bufs[1][0], bufs[2][0], bufs[3][0])
    torch.cuda.synchronize()
    for _, buf, guard in bufs:
        assert guards_intact(buf, guard)
    ax, aw, ag = np.abs(x), np.abs(w), np.abs(gy)
    pixels = gy.size // ws[0]
    _within("y", host(y), ref, f(ax, aw, np.abs(b)), fan)
    _within("dx", host(gx), dx(gy, w), dx(ag, aw), ws[0] * fan // ws[1])
    _within("dW", host(gw), dw(gy, x), dw(ag, ax), pixels)


@pytest.mark.parametrize("case", range(len(CHAINS)))
def test_f32_long_sums_run_in_short_chains(case):
    """Every product is p, whose low bits a partial sum of 2^e and more loses in
    the same direction at each addition: a chain of K products is off by up to
    K / 2 * 2^-24 of the sum, chains of 256 and their sum by at most (128 + K / 512
    + 8) * 2^-24 (half of each bound, as the partial sums grow from zero)."""
    pas, n, c, size, k, f, stride = CHAINS[case]
    terms = f * f * c if pas == "y" else (-(-f // stride)) ** 2 * k
    e = terms.bit_length() - (1 if terms >= 1.5 * 2 ** (terms.bit_length() - 1) else 2)
    p = 1 + 2.0 ** (e - 24) - 2.0 ** -22
    out = (size + 2 * (f // 2) - f) // stride + 1
    w = torch.ones(k, c, f, f, device="cuda").contiguous(memory_format=torch.channels_last)
    x = torch.full((n, c, size, size), p, device="cuda").contiguous(memory_format=torch.channels_last)
    y, rec = ms.layer_forward(ms.Conv2d(stride, f // 2), x, w, None, 1)
    if pas == "y":
        ones = np.ones((1, 1, size, size))
        count = c * oracle.conv2d_forward(ones, np.ones((1, 1, f, f)), None, (stride, stride), (f // 2, f // 2))
        got = y
    else:
        ones = np.ones((1, 1, out, out))
        count = k * oracle.conv2d_input_grad(ones, np.ones((1, 1, f, f)), (1, 1, size, size), (stride, stride), (f // 2, f // 2))
        got = ms.layer_backward(rec, torch.full_like(y, p))[0]
    assert count.max() == terms
    err = np.abs(host(got) - p * count).max() / (p * terms)
    assert err <= (128 + terms / 512 + 8) * 2.0 ** -24, err * 2.0 ** 24


def test_f32_transposed_convolution_bias_and_output_padding():
    xs, ws, stride, pad, op = (2, 32, 5, 6), (32, 34, 4, 3), (2, 3), (1, 1), (1, 2)
    x, w = synth.normal(xs, 9500, dtype="f32"), synth.kaiming_uniform(ws, 9501, 34 * 12, dtype="f32")
    b = synth.normal((34,), 9502, 1.0, dtype="f32")
    ref = oracle.convt2d_forward(x, w, b, stride, pad, op)
    y, _ = ms.layer_forward(ms.ConvTranspose2d(stride, pad, op), dev(x, "f32"), dev(w, "f32"), dev(b, "f32"), 0)
    _within("y", host(y), ref, oracle.convt2d_forward(np.abs(x), np.abs(w), np.abs(b), stride, pad, op), 32 * 12)


@pytest.mark.parametrize("xs,ws,stride,op", [
    ((16, 8, 101, 150), (8, 8, 3, 3), (1, 1), (0, 0)),    # whole output vectors
    ((6, 12, 99, 81), (12, 5, 4, 3), (2, 2), (1, 0)),     # strided phases, five output channels
])
def test_f32_few_channel_transposed_forward_with_bias(xs, ws, stride, op):
    """The few-channel input-gradient kernel with a bias: a transposed forward."""
    pad = (1, 1)
    x, w = synth.normal(xs, 9510, dtype="f32"), synth.kaiming_uniform(ws, 9511, ws[0] * ws[2] * ws[3], dtype="f32")
    b = synth.normal((ws[1],), 9512, 1.0, dtype="f32")
    ref = oracle.convt2d_forward(x, w, b, stride, pad, op)
    geom = (xs[0], ws[1], *ref.shape[2:], ws[0], *ws[2:], *xs[2:], *stride, *pad)
    plan = (C.c_int64 * 5)()
    assert _lib.load().ms_testing_float_plan(1, (C.c_int32 * 13)(*geom), plan) == 0 and plan[3] == 1
    out, buf, guard = guarded_empty(ref.shape, "f32")
    y, _ = ms.layer_forward(ms.ConvTranspose2d(stride, pad, op), dev(x, "f32"), dev(w, "f32"), dev(b, "f32"), 0, y=out)
    assert guards_intact(buf, guard)
    _within("y", host(y), ref, oracle.convt2d_forward(np.abs(x), np.abs(w), np.abs(b), stride, pad, op), ws[0] * ws[2] * ws[3])


@pytest.mark.parametrize("channels", [32, 6])
def test_f32_nonfinite_input_reaches_its_outputs_only(channels):
    """An infinite and a NaN pixel: outputs that read them are not finite (an
    infinity stays one where it meets no zero weight), the rest are as without."""
    xs, ws = (1, channels, 9, 9), (16, channels, 3, 3)
    x, w = synth.normal(xs, 9600, dtype="f32"), synth.kaiming_uniform(ws, 9601, 9 * channels, dtype="f32")
    clean = oracle.conv2d_forward(x, w, None, (1, 1), (1, 1))
    bad = x.copy()
    bad[0, 1, 2, 2], bad[0, 3, 6, 7] = np.inf, np.nan
    y, _ = ms.layer_forward(ms.Conv2d(1, 1), dev(bad, "f32"), dev(w, "f32"), None, 0)
    y = host(y)
    hit = np.zeros((9, 9), bool)
    hit[1:4, 1:4] = hit[5:8, 6:9] = True
    assert np.isinf(y[0, :, 1:4, 1:4]).all() and np.isnan(y[0, :, 5:8, 6:9]).all()
    _within("rest", np.where(hit, 0, y), np.where(hit, 0, clean),
            oracle.conv2d_forward(np.abs(x), np.abs(w), None, (1, 1), (1, 1)), 9 * channels)


def test_f32_few_channel_weight_gradient_keeps_infinities_apart():
    """An infinity of one input channel reaches that channel's weight gradients
    as an infinity, through ragged strips and ranges, and no other's."""
    xs, ws = (4, 8, 61, 300), (8, 8, 3, 3)
    x, gy = synth.normal(xs, 9700, dtype="f32"), synth.normal((4, 8, 61, 300), 9701, dtype="f32")
    for pixel in ((0, 30, 299), (1, 60, 287), (3, 0, 0), (2, 31, 150)):
        bad = x.copy()
        bad[pixel[0], 5, pixel[1], pixel[2]] = np.inf
        w = synth.kaiming_uniform(ws, 9702, 72, dtype="f32")
        _, rec = ms.layer_forward(ms.Conv2d(1, 1), dev(bad, "f32"), dev(w, "f32"), None, 2)
        _, gw, _ = ms.layer_backward(rec, dev(gy, "f32"))
        gw = host(gw)
        assert not np.isnan(gw).any() and np.isfinite(np.delete(gw, 5, 1)).all()
        assert np.isinf(gw[:, 5, 1, 1]).all()


def test_f32_passes_captured_without_workspace():
    """A capture on a stream that holds no workspace: the passes that would split
    their reduction for it run unsplit instead of allocating."""
    xs, ws = (1, 128, 4, 4), (256, 128, 3, 3)
    x, w = synth.normal(xs, 9700, dtype="f32"), synth.kaiming_uniform(ws, 9701, 1152, dtype="f32")
    gy = synth.normal((1, 256, 4, 4), 9702, dtype="f32")
    X, W, G = (dev(t, "f32") for t in (x, w, gy))

    def passes():
        y, rec = ms.layer_forward(ms.Conv2d(1, 1), X, W, None, 1)
        return y, ms.layer_backward(rec, G)[0]

    def right(y, dx):
        torch.cuda.synchronize()
        ax, aw, ag = np.abs(x), np.abs(w), np.abs(gy)
        _within("y", host(y), oracle.conv2d_forward(x, w, None, (1, 1), (1, 1)),
                oracle.conv2d_forward(ax, aw, None, (1, 1), (1, 1)), 1152)
        _within("dx", host(dx), oracle.conv2d_input_grad(gy, w, xs, (1, 1), (1, 1)),
                oracle.conv2d_input_grad(ag, aw, xs, (1, 1), (1, 1)), 2304)

    right(*passes())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        got = passes()
    for _ in range(3):
        for t in got:
            t.fill_(float("nan"))
        graph.replay()
        right(*got)
        right(*passes())


@pytest.mark.parametrize("dtype,channels", [("f32", (128, 256)), ("bf16", (60, 100))])
def test_captured_passes_hold_no_workspace(dtype, channels):
    """An input gradient captured on a stream whose workspace would do: the graph
    holds none of it (fp32 runs unsplit, ragged bf16 channels as with no room for
    copies), so the stream may outgrow it and replays stay as they were."""
    c, k = channels
    xs, ws = (1, c, 4, 4), (k, c, 3, 3)
    x, w = synth.normal(xs, 9710, dtype=dtype), synth.kaiming_uniform(ws, 9711, 9 * c, dtype=dtype)
    X, W, G = (dev(t, dtype) for t in (x, w, synth.normal((1, k, 4, 4), 9712, dtype=dtype)))
    lib = _lib.load()
    recs = [ms.layer_forward(ms.Conv2d(1, 1), X, W, None, 1)[1] for _ in range(3)]
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):   # one that has no workspace yet
        lib.ms_testing_fail_next_workspace(1)
        without = ms.layer_backward(recs[0], G)[0]
        lib.ms_testing_fail_next_workspace(0)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        ms.layer_backward(recs[1], G)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        got = ms.layer_backward(recs[2], G)[0]
    big, bw = (torch.randn(s, device="cuda", dtype=X.dtype) for s in ((2048, 4095), (1023, 4095)))
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        _, rec = ms.layer_forward(ms.Linear(), big, bw, None, 2)
        ms.layer_backward(rec, torch.ones(2048, 1023, device="cuda", dtype=X.dtype))
    torch.cuda.synchronize()
    spare = [torch.full((1 << 19,), 3.0, device="cuda") for _ in range(8)]
    for _ in range(3):
        got.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, without)
        assert all(bool((t == 3.0).all()) for t in spare)


def test_outgrown_workspace_of_a_graph_is_kept():
    """A bf16 forward on padded copies holds the stream's workspace in its graph:
    a larger call on the stream does not free what replays write."""
    x, w = synth.normal((2, 60, 9, 9), 9720, dtype="bf16"), synth.kaiming_uniform((64, 60, 3, 3), 9721, 540, dtype="bf16")
    X, W = dev(x, "bf16"), dev(w, "bf16")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        want, _ = ms.layer_forward(ms.Conv2d(1, 1), X, W, None, 0)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        got, _ = ms.layer_forward(ms.Conv2d(1, 1), X, W, None, 0)
    big, bw = torch.randn(8192, 1023, device="cuda").bfloat16(), torch.randn(256, 1023, device="cuda").bfloat16()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        ms.layer_forward(ms.Linear(), big, bw, None, 0)
    torch.cuda.synchronize()
    spare = [torch.full((1 << 19,), 3.0, device="cuda") for _ in range(8)]
    for _ in range(3):
        got.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        assert all(bool((t == 3.0).all()) for t in spare)
