"""bf16 weight and bias gradients whose reduction is split many ways over a small
output, so that thread groups share the sum of the partials: row counts that the
planner splits 7 to 16 ways, outputs that end inside a block's columns, channels
cropped from padded rows, and the output from which no groups share.

Bar: one rounding to bf16 (2^-8 of the value) and, for K products summed in
fp32, K * 2^-24 of the sum of their magnitudes."""
import pytest
import torch

import paper_2404_12406_amd as ms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1927, 2500, 2563, 4099, 4611, 16899])
@pytest.mark.parametrize("channels", [(8, 8), (12, 10), (64, 72), (130, 257), (512, 504), (512, 520)])
def test_split_gradient_sums(channels, m):
    k, n = channels
    g = torch.Generator(device="cuda").manual_seed(1000 * n + m)
    x, dy = (torch.randn(m, c, generator=g, device="cuda").bfloat16() for c in (k, n))
    w, b = (torch.randn(s, generator=g, device="cuda").bfloat16() for s in ((n, k), (n,)))
    _, rec = ms.layer_forward(ms.Linear(), x, w, b, ms.MASK_WEIGHT | ms.MASK_BIAS)
    _, gw, gb = ms.layer_backward(rec, dy)
    X, D = x.double(), dy.double()
    for name, got, ref, mag in (("dW", gw, D.t() @ X, D.abs().t() @ X.abs()), ("db", gb, D.sum(0), D.abs().sum(0))):
        bad = (got.double() - ref).abs() - (2.0 ** -8 * ref.abs() + (m + 8) * 2.0 ** -24 * mag)
        assert bool(torch.isfinite(got).all()) and float(bad.max()) <= 0, (name, float(bad.max()))
