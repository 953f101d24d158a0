"""From 3072 groups of more than 2048 elements on, a wavefront takes each: where that begins, one group more must not cost a jump in
time, whatever the method and the data, since the choice sees neither.  And bit for bit with the oracle there."""
import pytest
import torch

import paper_2508_00806_amd as adacc
from helpers import run_parity

pytestmark = pytest.mark.gpu

GROUPS = 3072  # from here on a wavefront per group


def microseconds(m, n, xs):
    """The fastest of several runs of compressions of the first n elements of each tensor in turn."""
    blobs = [adacc.alloc_blob(m, n)[0] for _ in xs]
    ws = adacc.alloc_workspace(adacc.workspace_bytes(m, n))
    views = [x[:n] for x in xs]
    begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for run in range(8):
        begin.record()
        for i in range(20):
            adacc.compress(m, views[i % len(xs)], blobs[i % len(xs)], ws)
        end.record()
        torch.cuda.synchronize()
        best = min(best, begin.elapsed_time(end) / 20 * 1e3) if run else best
    return best


def values(kind, gs, dtype=torch.bfloat16):
    g = torch.Generator(device="cuda").manual_seed(gs)
    x = torch.nn.functional.silu(torch.randn(GROUPS, gs, generator=g, device="cuda") * 1.5)
    return x.to(dtype).view(-1)


def check_line(kind, gs, gq, k):
    """Measured: at most 1.05 where the wavefronts are right, 1.4 and more where they were not."""
    xs = [values(kind, gs) for _ in range(4)]
    m = adacc.Method(bits=4, quant_group=gq, outlier_mode=adacc.OUTLIER_TOPK, stat_group=gs, topk=k, max_outliers=GROUPS * gs // 8)
    few, many = (microseconds(m, n * gs, xs) for n in (GROUPS - 1, GROUPS))
    print(f"[line] {kind} gs={gs} k={k}: {GROUPS - 1} groups {few:.1f} us, {GROUPS} {many:.1f}", flush=True)
    assert many < 1.2 * few


@pytest.mark.parametrize("gs,gq", [(2200, 2200), (4096 - 8, 8)])
@pytest.mark.parametrize("k", [9, 32])
def test_many_of_the_largest(gs, gq, k):
    check_line("silu", gs, gq, k)


@pytest.mark.parametrize("end", [8, 24, 2048])
@pytest.mark.parametrize("k", [9, 32])
def test_many_of_the_largest_against_the_oracle(end, k):
    """.. with the tensor's last group short, of fewer elements than k too."""
    gs = 2560
    x = torch.nn.functional.silu(torch.randn(GROUPS * gs + end, generator=torch.Generator().manual_seed(end)) * 1.5)
    x.view(-1)[:gs] = 1.25
    print(f"[line] k={k} end={end}", flush=True)
    run_parity(x.to(torch.bfloat16), dict(bits=8, quant_group=128, asym=1, outlier_mode="topk", stat_group=gs, thresh=0.0, topk=k))
