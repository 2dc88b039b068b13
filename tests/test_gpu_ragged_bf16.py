"""bf16 gradients of layers whose channel counts are not multiples of 8, which
run on padded copies of dy and x with the filter transposed element by element:
each remainder of 8 on either side, whole reduction steps and not, strided
phases, the narrow kernels for 64 channels, a stem's packed input, split and
unsplit, misaligned tensors, the transposed layer's bias, and a scratch too
small for the copies.

Bar: one rounding to bf16 (2^-8 of the value) and, for K products summed in
fp32, K * 2^-24 of the sum of their magnitudes."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import paper_2404_12406_amd as ms
import synth
from paper_2404_12406_amd import _lib, api

from _gpu import dev, guarded_empty, guards_intact, host

pytestmark = pytest.mark.gpu


def _within(name, got, ref, magnitude, k):
    bad = np.abs(got - ref) - (2.0 ** -8 * np.abs(ref) + (k + 8) * 2.0 ** -24 * magnitude)
    assert np.isfinite(got).all() and bad.max() <= 0, (name, float(np.abs(got - ref).max()), float(bad.max()))


CASES = [
    # x, w, stride, pad, guard elements before the outputs (64: aligned)
    ((3, 60, 13, 11), (100, 60, 3, 3), (2, 2), (1, 1), 64),     # ragged both ways, strided phases
    ((3, 60, 13, 11), (100, 60, 3, 3), (2, 2), (1, 1), 65),     # outputs off alignment
    ((2, 64, 12, 9), (57, 64, 3, 3), (1, 1), (1, 1), 64),       # dy padded to 64 channels, whole vectors of dx
    ((2, 61, 12, 9), (60, 61, 3, 3), (1, 1), (1, 1), 64),       # and dx cropped from 64
    ((2, 62, 12, 10), (63, 62, 3, 3), (2, 2), (1, 1), 64),      # the same through output phases
    ((2, 33, 9, 8), (127, 33, 3, 3), (1, 1), (1, 1), 64),       # whole steps of the padded reduction
    ((1, 130, 5, 5), (513, 130, 3, 3), (1, 1), (1, 1), 64),     # a deep reduction of few tiles: split
    ((9, 1, 17, 15), (1, 1, 5, 5), (1, 1), (2, 2), 64),         # one channel each way
    ((2, 3, 33, 31), (30, 3, 7, 7), (2, 2), (3, 3), 64),        # a stem with ragged filters
    ((2, 3, 33, 31), (64, 3, 7, 7), (2, 2), (3, 3), 64),        # and with whole ones
    ((5, 12, 30, 31), (20, 12, 2, 3), (1, 3), (0, 1), 64),      # uneven strides: phases without taps
    ((1030, 131), (333, 131), None, None, 64),                  # fully connected, odd both ways
    ((259, 515), (1001, 515), None, None, 65),
    ((4099, 12), (10, 12), None, None, 64),                     # a long reduction of one tile
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_ragged_gradients(case):
    xs, ws, stride, pad, guard = CASES[case]
    seed, fan = 12000 + 10 * case, int(np.prod(ws[1:]))
    x = synth.normal(xs, seed, dtype="bf16")
    w = synth.kaiming_uniform(ws, seed + 1, fan, dtype="bf16")
    b = synth.normal((ws[0],), seed + 2, 1.0, dtype="bf16")
    if stride is None:
        spec = ms.Linear()
        f, dx, dw = oracle.linear_forward, lambda g, w: oracle.linear_input_grad(g, w), lambda g, x: oracle.linear_weight_grad(g, x)
    else:
        spec = ms.Conv2d(stride, pad)
        f = lambda x, w, b: oracle.conv2d_forward(x, w, b, stride, pad)
        dx = lambda g, w: oracle.conv2d_input_grad(g, w, xs, stride, pad)
        dw = lambda g, x: oracle.conv2d_weight_grad(g, x, ws, stride, pad)
    ref = f(x, w, b)
    gy = synth.normal(ref.shape, seed + 3, dtype="bf16")
    bufs = [guarded_empty(s, "bf16", guard) for s in (xs, ws, (ws[0],))]
    y, rec = ms.layer_forward(spec, dev(x, "bf16"), dev(w, "bf16"), dev(b, "bf16"), 7)
    gx, gw, gb = ms.layer_backward(rec, dev(gy, "bf16"), bufs[0][0], bufs[1][0], bufs[2][0])
    torch.cuda.synchronize()
    for _, buf, guard in bufs:
        assert guards_intact(buf, guard)
    ax, aw, ag = np.abs(x), np.abs(w), np.abs(gy)
    pixels = gy.size // ws[0]
    _within("y", host(y), ref, f(ax, aw, np.abs(b)), fan)
    _within("dx", host(gx), dx(gy, w), dx(ag, aw), ws[0] * fan // ws[1])
    _within("dW", host(gw), dw(gy, x), dw(ag, ax), pixels)
    axes = (0,) + tuple(range(2, gy.ndim))
    _within("db", host(gb), gy.astype(np.float64).sum(axes), ag.astype(np.float64).sum(axes), pixels)


@pytest.mark.parametrize("channels", [(60, 60), (33, 21)])
def test_ragged_transposed_forward_with_bias(channels):
    k, c = channels
    xs, ws, stride, pad, op = (2, k, 9, 7), (k, c, 3, 3), (2, 2), (1, 1), (1, 1)
    x, w = synth.normal(xs, 12500, dtype="bf16"), synth.kaiming_uniform(ws, 12501, 9 * c, dtype="bf16")
    b = synth.normal((c,), 12502, 1.0, dtype="bf16")
    ref = oracle.convt2d_forward(x, w, b, stride, pad, op)
    y, _ = ms.layer_forward(ms.ConvTranspose2d(stride, pad, op), dev(x, "bf16"), dev(w, "bf16"), dev(b, "bf16"), 0)
    _within("y", host(y), ref, oracle.convt2d_forward(np.abs(x), np.abs(w), np.abs(b), stride, pad, op), 9 * k)


def test_ragged_nonfinite_dy_reaches_its_gradients_only():
    """The padded products are zeros times zeros: an infinite and a NaN element
    of dy leave the gradients of other pixels and filters alone."""
    xs, ws = (1, 20, 9, 9), (21, 20, 3, 3)
    x, w = synth.normal(xs, 12600, dtype="bf16"), synth.kaiming_uniform(ws, 12601, 180, dtype="bf16")
    gy = synth.normal((1, 21, 9, 9), 12602, dtype="bf16")
    gy[0, 2, 2, 2], gy[0, 20, 6, 7] = np.inf, np.nan
    y, rec = ms.layer_forward(ms.Conv2d(1, 1), dev(x, "bf16"), dev(w, "bf16"), None, 3)
    gx, gw, _ = ms.layer_backward(rec, dev(gy, "bf16"))
    near = np.zeros((9, 9), bool)
    near[1:4, 1:4] = near[5:8, 6:9] = True
    assert np.isfinite(host(gx)[0][:, ~near]).all() and not np.isfinite(host(gx)[0][:, near]).any()
    hit = np.zeros(21, bool)
    hit[[2, 20]] = True
    assert np.isfinite(host(gw)[~hit]).all() and not np.isfinite(host(gw)[20]).any()


def test_ragged_noalloc_without_room_for_the_copies():
    """A padded dy larger than the fixed scratch: the gradients run without it."""
    m, k, n = 600000, 16, 60
    g = torch.Generator(device="cuda").manual_seed(5)
    x, dy = (torch.randn(m, c, generator=g, device="cuda").bfloat16() for c in (k, n))
    w = torch.randn(n, k, generator=g, device="cuda").bfloat16()
    lib = _lib.load()
    assert m * 64 * 2 > lib.ms_noalloc_scratch_bytes()
    _, rec = ms.layer_forward(ms.Linear(), x, w, None, 3)
    gx, gw = torch.empty_like(x), torch.empty_like(w)
    d = [api.tensor_desc(t) for t in (dy, gx, gw)]
    torch.cuda.synchronize()
    st = lib.ms_layer_backward_noalloc(rec._h, C.byref(d[0]), C.byref(d[1]), C.byref(d[2]), None, api._stream(x.device))
    torch.cuda.synchronize()
    assert st == _lib.MS_OK
    for name, got, a, b, terms in (("dx", gx, dy, w, n), ("dW", gw, dy.t(), x, m)):
        ref, mag = a.double() @ b.double(), a.double().abs() @ b.double().abs()
        _within(name, host(got), ref.cpu().numpy(), mag.cpu().numpy(), terms)
