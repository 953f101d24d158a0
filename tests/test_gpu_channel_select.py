"""The selection of outlier channels by Z-score: numbers of channels around what the threads keep in registers, thresholds below and at
zero, and channels whose Z is the threshold itself, which only the division of the definition decides."""
import numpy as np
import pytest
import torch

import paper_2508_00806_amd as adacc
from helpers import run_channel_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden", [8, 16, 512, 4096, 4104, 8192, 8200, 12288, 65536])
@pytest.mark.parametrize("z", [2.5, 0.0, -0.25])
def test_numbers_of_channels(hidden, z):
    g = torch.Generator().manual_seed(hidden)
    x = torch.randn(16, hidden, generator=g).sign()  # every sum is exact
    at = torch.randperm(hidden, generator=g)[:max(1, hidden // 50)]
    x[:, at] *= 64.0
    x[:, hidden // 2] *= 3.0
    if hidden > 512:
        x[3, 77] = float("inf")
    print(f"[channel select] hidden={hidden} z={z}", flush=True)
    run_channel_parity(x.to(torch.bfloat16), 8, 8, 0, z=z)


@pytest.mark.parametrize("hidden", [16, 4096, 16384])
def test_a_score_that_is_the_threshold(hidden):
    """Half of the channels sum to 16, half to 48: mean 32, deviation 16, every Z exactly 1 or -1."""
    x = torch.ones(16, hidden)
    x[:, 1::2] = 3.0
    x = x.to(torch.bfloat16).cuda()
    for z, n in ((1.0, 0), (float(np.nextafter(np.float32(1.0), np.float32(0.0))), hidden // 2), (-1.0, hidden // 2),
                 (float(np.nextafter(np.float32(-1.0), np.float32(-2.0))), hidden)):
        m = adacc.ChannelMethod(bits=8, quant_group=8, z_thresh=z, max_channels=hidden)
        blob, L = adacc.alloc_channel_blob(m, 16, hidden)
        print(f"[channel select] hidden={hidden} z={z!r}", flush=True)
        adacc.channel_compress(m, x, 16, hidden, blob, adacc.alloc_channel_workspace(16, hidden))
        assert adacc.channel_read_status(blob, L) == (n, 0, 0, 0)
    flat = torch.ones(16, hidden, dtype=torch.bfloat16, device="cuda")  # deviation zero: Z is not a number
    for z in (3.0, 0.0, -3.0):
        m = adacc.ChannelMethod(bits=8, quant_group=8, z_thresh=z, max_channels=hidden)
        blob, L = adacc.alloc_channel_blob(m, 16, hidden)
        adacc.channel_compress(m, flat, 16, hidden, blob, adacc.alloc_channel_workspace(16, hidden))
        assert adacc.channel_read_status(blob, L) == (0, 0, 0, 0)
