"""Staging of plane-by-plane tensors with few channels: the staged call's
output is bit for bit that of the same values handed over channels-last, for
every channel count around the register copy's limit, whole and odd pixel
counts, batches of strided slices and bases off every alignment."""
import pytest
import torch

import paper_2404_12406_amd as ms

pytestmark = pytest.mark.gpu

DTYPES = [torch.float32, torch.bfloat16]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("channels", [1, 2, 3, 4, 5, 7, 8, 12, 15, 16, 17])
@pytest.mark.parametrize("hw", [(64, 48), (33, 35), (40, 30), (1, 2051)])
def test_planes_match_channels_last(dtype, channels, hw):
    g = torch.Generator(device="cuda").manual_seed(channels * 1000 + hw[0])
    full = torch.randn((3, channels + 2, *hw), generator=g, device="cuda").to(dtype)
    flat = torch.randn(2 * channels * hw[0] * hw[1] + 1, generator=g, device="cuda").to(dtype)
    for x in (full[:, :channels].contiguous(), full[:, 1:channels + 1], full[1:2, :channels],
              flat[1:].view(2, channels, *hw), full[:, :channels, :, 1:]):
        want, _ = ms.layer_forward(ms.AvgPool(), x.contiguous(memory_format=torch.channels_last))
        got, _ = ms.layer_forward(ms.AvgPool(), x)
        assert torch.equal(got, want)
