"""bf16 3-D convolutions whose depth taps run as further taps of the GEMM's
loads (no depth folding), at the edges of that path: whole reduction steps in
one tap and not, 32 taps and one more, strided depths, heights and widths,
images smaller than a pixel step, samples of few depths, 64 rows and 32 columns
and more, tensors off 16-byte alignment (which fold).

Bar: one rounding to bf16 (2^-8 of the value) and, for K products summed in
fp32, K * 2^-24 of the sum of their magnitudes."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_12406_amd as ms
import synth

from _gpu import host

pytestmark = pytest.mark.gpu


def _dev(a, offset=0):
    """Channels-last bf16 tensor starting `offset` elements into its storage."""
    t = torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(torch.bfloat16).cuda()
    if t.dim() == 5:
        t = t.contiguous(memory_format=torch.channels_last_3d)
    if not offset:
        return t
    buf = torch.empty(t.numel() + offset, dtype=t.dtype, device="cuda")
    v = buf.as_strided(t.shape, t.stride(), offset)
    v.copy_(t)
    return v


def _within(name, got, ref, magnitude, k):
    bad = np.abs(got - ref) - (2.0 ** -8 * np.abs(ref) + (k + 8) * 2.0 ** -24 * magnitude)
    assert np.isfinite(got).all() and bad.max() <= 0, (name, float(np.abs(got - ref).max()), float(bad.max()))


CASES = [
    # x, w, stride, pad, storage offset
    ((2, 64, 5, 9, 10), (64, 64, 3, 3, 3), (1, 1, 1), (1, 1, 1), 0),      # every pass, 64 rows / 64 columns
    ((2, 64, 6, 7, 5), (72, 64, 3, 3, 3), (2, 1, 1), (1, 1, 1), 0),       # depth stride: the input gradient folds
    ((1, 128, 4, 8, 9), (64, 128, 3, 3, 3), (1, 2, 2), (1, 1, 1), 0),     # strided height and width phases
    ((5, 64, 3, 2, 3), (128, 64, 3, 3, 3), (1, 1, 1), (1, 1, 1), 0),      # images of 6 pixels: several a step
    ((3, 64, 1, 1, 1), (64, 64, 3, 1, 1), (1, 1, 1), (1, 0, 0), 0),       # one pixel, one depth
    ((2, 24, 7, 6, 7), (64, 24, 2, 3, 3), (1, 1, 1), (0, 1, 1), 0),       # 24 input channels: 32-column tile, ragged
    ((2, 8, 9, 11, 6), (8, 8, 3, 3, 3), (3, 1, 1), (2, 1, 1), 0),         # weight gradient alone, deep stride and pad
    ((1, 64, 5, 9, 9), (64, 64, 2, 4, 4), (1, 1, 1), (1, 2, 2), 0),       # 32 taps
    ((1, 64, 5, 7, 7), (64, 64, 3, 4, 3), (1, 1, 1), (1, 2, 1), 0),       # 36 taps: folds, weight gradient does not
    ((2, 64, 9, 20, 21), (200, 64, 1, 1, 1), (1, 1, 1), (0, 0, 0), 0),    # pointwise
    ((2, 64, 5, 9, 10), (64, 64, 3, 3, 3), (1, 1, 1), (1, 1, 1), 1),      # off alignment: folds
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_conv3d_taps(case):
    xs, ws, stride, pad, off = CASES[case]
    seed, fan = 9800 + 10 * case, int(np.prod(ws[1:]))
    x = synth.normal(xs, seed, dtype="bf16")
    w = synth.kaiming_uniform(ws, seed + 1, fan, dtype="bf16")
    b = synth.normal((ws[0],), seed + 2, 1.0, dtype="bf16")
    ref = oracle.conv3d_forward(x, w, b, stride, pad)
    gy = synth.normal(ref.shape, seed + 3, dtype="bf16")
    y, rec = ms.layer_forward(ms.Conv3d(stride, pad), _dev(x, off), _dev(w, off), _dev(b), 7)
    gx, gw, gb = ms.layer_backward(rec, _dev(gy, off))
    ax, aw, ag = np.abs(x), np.abs(w), np.abs(gy)
    folds = off or ws[2] * ws[3] * ws[4] > 32 or stride[0] > 1
    _within("y", host(y), ref, oracle.conv3d_forward(ax, aw, np.abs(b), stride, pad), fan)
    # a folded input gradient rounds each depth tap's sum before adding them
    mag = oracle.conv3d_input_grad(ag, aw, xs, stride, pad)
    _within("dx", host(gx), oracle.conv3d_input_grad(gy, w, xs, stride, pad), mag,
            ws[0] * fan // ws[1] + (2 ** 15 if folds or ws[0] % 64 else 0))
    _within("dW", host(gw), oracle.conv3d_weight_grad(gy, x, ws, stride, pad),
            oracle.conv3d_weight_grad(ag, ax, ws, stride, pad), gy.size // ws[0])
    _within("db", host(gb), oracle.bias_grad5(gy), oracle.bias_grad5(ag), gy.size // ws[0])


def test_conv3d_transpose_taps_with_bias():
    """Its forward is the input-gradient contraction with a bias, at unit depth
    step and strided height and width."""
    xs, ws, stride, pad, op = (2, 64, 4, 5, 6), (64, 16, 3, 4, 4), (1, 2, 2), (1, 1, 1), (0, 1, 0)
    x, w = synth.normal(xs, 9950, dtype="bf16"), synth.kaiming_uniform(ws, 9951, 16 * 48, dtype="bf16")
    b = synth.normal((16,), 9952, 1.0, dtype="bf16")
    ref = oracle.convt3d_forward(x, w, b, stride, pad, op)
    y, _ = ms.layer_forward(ms.ConvTranspose3d(stride, pad, op), _dev(x), _dev(w), _dev(b), 0)
    _within("y", host(y), ref, oracle.convt3d_forward(np.abs(x), np.abs(w), np.abs(b), stride, pad, op), 64 * 48)
