"""The places of the outliers in the stream: tiles at and beyond what a slot of the workspace holds, short tensors (every
workgroup adds up all counts before its own) and long ones (sums of blocks first), tiles and the fallback kernels'
segments, and the end that the groups do not divide, with outliers of its own."""
import pytest
import torch

from helpers import run_parity

pytestmark = pytest.mark.gpu

# (quantisation group, elements of a tile, whole tiles, elements behind them)
SHAPES = [(64, 2048, 64, 63), (64, 2048, 65, 0), (4096, 4096, 9, 4095), (512, 2048, 0, 511), (40, 4080, 17, 1001), (11008, 11008, 16, 0),
          (64, 2048, 32768 + 260, 33), (40, 4080, 32768 + 17, 9)]


@pytest.mark.parametrize("gq,tile,tiles,rest", SHAPES)
def test_slots_at_their_limit(gq, tile, tiles, rest):
    n = tile * tiles + rest
    g = torch.Generator().manual_seed(n)
    x = (torch.rand(n, generator=g) - 0.5).to(torch.bfloat16)
    # 63, 64, 65 outliers and a tile full of them, at both ends and across the workgroups' and sums' blocks
    for t, k in ((0, 64), (1, 65), (3, 63), (7, tile), (8, 1), (15, 65), (16, 64), (63, 64), (64, 65), (255, 70), (256, 3), (32767, 65),
                 (32768, 64), (tiles - 1, 65)):
        if 0 <= t < tiles:
            at = t * tile + torch.randperm(tile, generator=g)[:k]
            x[at] = 2.0 + torch.rand(k, generator=g).to(torch.bfloat16)
    if rest:
        x[n - rest:n - rest + 3] = -3.0
        x[n - 1] = float("inf")
    print(f"[placement] gq={gq} tiles={tiles} rest={rest}", flush=True)
    oc, *_ = run_parity(x, dict(bits=8, quant_group=gq, asym=0, outlier_mode="abs", stat_group=0, thresh=1.0, topk=0))
    assert oc.n_out > 0


@pytest.mark.parametrize("mode", ["none", "abs", "std", "topk"])
@pytest.mark.parametrize("rest", [1, 8, 1999, 2048, 2049, 4095])
def test_the_end_of_a_tensor_that_its_groups_do_not_divide(mode, rest):
    for gq, gs, bits, asym, dtype in ((64, 4096, 4, 0, torch.bfloat16), (4096, 4096, 8, 1, torch.float16), (4096, 4096, 4, 0, torch.bfloat16)):
        for whole in (0, 4096):
            x = torch.randn(whole + rest, generator=torch.Generator().manual_seed(rest)).to(dtype)
            x[-1] = float("nan")
            print(f"[end] {mode} rest={rest} gq={gq} bits={bits} asym={asym} whole={whole}", flush=True)
            run_parity(x, dict(bits=bits, quant_group=gq, asym=asym, outlier_mode=mode, stat_group=gs,
                               thresh=2.0 if mode in ("abs", "std") else 0.0, topk=7 if mode == "topk" else 0))


# a workgroup of the placement takes 1, 2, 4, 8, 16 segments of the fallback kernels, TOPK of very many several times 16
SEGMENTS = ([("std", 2056, s) for s in (1, 5, 1024, 1025, 2049, 4097, 8193, 32769 + 15)] +
            [("topk", 2056, s) for s in (1, 5, 4096, 4097, 16385, 65537 + 21)] + [("topk", 4104, s) for s in (1025, 16385 + 18)])


@pytest.mark.parametrize("mode,group,segments", SEGMENTS)
def test_segments_selected_again(mode, group, segments):
    """Some segments beyond their slot (STD), all of them once more because one is irregular (TOPK)."""
    n = group * segments - 700
    g = torch.Generator().manual_seed(segments)
    x = (torch.rand(n, generator=g) - 0.5).to(torch.bfloat16)
    at = {0, segments // 2, max(segments - 2, 0), segments - 1} | set(range(3, min(segments, 40), 5))
    for t in at:
        first = group * t
        k = min(70 + t % 7, n - first)
        x[first:first + k] = 9.0 + (torch.arange(k) % 5).to(torch.bfloat16)
    if mode == "topk":
        x[group * (segments // 2) + 100:group * (segments // 2) + 105] = float("inf")
    print(f"[placement] {segments} segments of {group}, {mode}", flush=True)
    oc, *_ = run_parity(x, dict(bits=8, quant_group=group, asym=0, outlier_mode=mode, stat_group=group, thresh=2.0, topk=2))
    assert oc.n_out > (64 if mode == "std" else 2 * segments)


@pytest.mark.parametrize("group", [24, 504, 512 + 8, 1000, 2040])
def test_topk_groups_of_the_fallback_kernels(group):
    """Short and long groups have kernels of their own; regular, and with a group that has more infinities than k."""
    for extra in (0, 9):
        for k in (1, 5):
            n = group * 41 - 13
            x = torch.randn(n, generator=torch.Generator().manual_seed(group + k)).to(torch.float16)
            x[7 * group:7 * group + extra] = float("inf")
            print(f"[placement] topk {k} of {group}, {extra} infinities", flush=True)
            run_parity(x, dict(bits=4, quant_group=group, asym=1, outlier_mode="topk", stat_group=group, thresh=0.0, topk=k))


@pytest.mark.parametrize("tiles,rest", [(32768, 0), (32768 + 261, 1999)])
def test_long_topk_tensor_with_irregular_groups(tiles, rest):
    """Where a workgroup of the placement begins to take 256 tiles: groups with more infinities than k next to its borders."""
    n = 2048 * tiles + rest
    x = (torch.rand(n, generator=torch.Generator().manual_seed(tiles)) - 0.5).to(torch.bfloat16)
    for t in (0, 63, 64, 255, 256, 257, 32767, tiles - 1):
        x[2048 * t + 5:2048 * t + 9 + t % 3] = float("-inf")
    print(f"[placement] topk, {tiles} tiles", flush=True)
    oc, *_ = run_parity(x, dict(bits=4, quant_group=128, asym=0, outlier_mode="topk", stat_group=2048, thresh=0.0, topk=2))
    assert oc.n_out > 2 * tiles
