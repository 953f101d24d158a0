"""Outlier channels of few tokens: with and without the kernel that adds up the chunk sums, on both sides of its line."""
import pytest
import torch

from helpers import run_channel_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens", [8, 64, 65, 129, 192, 256, 257, 320])
@pytest.mark.parametrize("hidden", [8, 768, 4104, 8192, 8200])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_few_tokens(tokens, hidden, dtype):
    g = torch.Generator().manual_seed(tokens * hidden)
    x = torch.randn((tokens // 8 * 8 if hidden % 64 else tokens, hidden), generator=g)
    x[:, torch.randperm(hidden, generator=g)[:max(1, hidden // 300)]] *= 25.0
    if hidden > 8:
        x[3, 5] = float("inf")
    print(f"[few tokens] {tuple(x.shape)} {dtype}", flush=True)
    run_channel_parity(x.to(dtype), 4, 64 if x.numel() % 64 == 0 else 8, 0)
