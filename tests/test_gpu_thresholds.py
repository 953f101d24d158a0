"""ABS and STD through a threshold on the 16-bit magnitude, and TOPK over groups of two rows of a tile: group sizes of both kinds
on every side of a 512-element row, limits that fall on a representable square, limits so small that squares underflow, limits that
overflow, several outliers in one octet, all elements of a row, values that are not finite, a last tile that is not complete.
Every result is compared with the oracle bit for bit."""
import numpy as np
import pytest
import torch

from helpers import run_parity

pytestmark = pytest.mark.gpu

SIZES = [(32, 64), (64, 256), (8, 512), (64, 512), (512, 1024), (1024, 1024), (256, 2048), (2048, 2048), (128, 4096), (1024, 4096),
         (4096, 4096)]


def tensor(gs, g, dtype):
    """Eleven statistics groups of different kinds and half of a tile."""
    n = max(gs, 16)
    out = []
    for kind in ("normal", "octet", "constant", "pairs", "tiny", "tinier", "huge", "inf", "nan", "zeros", "negative"):
        x = torch.randn(n, generator=g)
        if kind == "octet":
            x[8:16] = torch.tensor([50.0, -60.0, 0.0, 70.0, 80.0, -90.0, 55.0, 65.0])
        elif kind == "constant":
            x[:] = 1.25
        elif kind == "pairs":  # two magnitudes, powers of two: the limit is a square or next to one
            x = torch.where(x > 1.0, 4.0, 2.0)
        elif kind == "tiny":
            x *= 1e-19  # bf16: squares around the smallest normal binary32
        elif kind == "tinier":
            x *= 1e-22  # squares subnormal and zero
        elif kind == "huge":
            x *= 3e18 if dtype == torch.bfloat16 else 2e4  # squares near the end of binary32
        elif kind == "inf":
            x[::n // 4] = float("inf")
        elif kind == "nan":
            x[3] = float("nan")
            x[n - 1] = float("-inf")
        elif kind == "zeros":
            x[:] = -0.0
            x[n // 2] = 1.0
        elif kind == "negative":
            x = -x.abs()
        out.append(x)
    return torch.cat(out + [torch.randn(1024, generator=g)]).to(dtype)


@pytest.mark.parametrize("mode,par", [("std", 2.0), ("std", 0.0), ("std", 5.0), ("abs", 2.0), ("abs", 0.0), ("abs", 1e30), ("none", 0.0),
                                      ("topk", 1), ("topk", 3), ("topk", 9)])
@pytest.mark.parametrize("gq,gs", SIZES)
def test_outliers_of_every_group_size(gq, gs, mode, par):
    g = torch.Generator().manual_seed(gq * gs)
    for dtype in (torch.bfloat16, torch.float16):
        x = tensor(gs, g, dtype)
        for bits, asym in ((8, 0), (4, 1)):
            print(f"[thresholds] {mode} {par} gq={gq} gs={gs} {dtype} int{bits} asym={asym}", flush=True)
            run_parity(x, dict(bits=bits, quant_group=gq, asym=asym, outlier_mode=mode, stat_group=gs if mode in ("std", "topk") else 0,
                               thresh=float(par) if mode in ("std", "abs") else 0.0, topk=par if mode == "topk" else 0))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
def test_thresholds_at_every_magnitude(dtype):
    """ABS with tau at, just below and just above magnitudes of the whole range of the format (all finite patterns are in the tensor)."""
    end = 0x7F80 if dtype == torch.bfloat16 else 0x7C00
    x = torch.arange(end, dtype=torch.int32).to(torch.int16).view(dtype)
    x = torch.cat([x, -x[: 2048 - end % 2048 + 77]])
    vals = x[:end].to(torch.float32).numpy()
    rng = np.random.default_rng(1)
    for m in [0, 1, 2, 0x7F, 0x80, 0x400, end - 2, end - 1] + list(rng.integers(3, end - 2, 12)):
        for tau in (vals[m], np.nextafter(vals[m], np.float32(-1.0), dtype=np.float32), np.nextafter(vals[m], np.float32(np.inf), dtype=np.float32)):
            if not (tau >= 0.0 and np.isfinite(tau)):
                continue
            print(f"[tau] pattern {m:#x} tau={tau!r} {dtype}", flush=True)
            run_parity(x, dict(bits=8, quant_group=1024, asym=0, outlier_mode="abs", stat_group=0, thresh=float(tau), topk=0), decompress=False)
