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
    if kind == "quarters":
        x = (x * 4).round() / 4
    elif kind == "eighths":  # three bits of significand
        x = torch.ldexp((torch.frexp(x)[0] * 16).round() / 16, torch.frexp(x)[1])
    elif kind == "clipped":
        x = x.clamp(max=2.0)
    elif kind == "equals":
        x[:, ::50] = 9.0
        x[:, 3] = 11.0
    elif kind == "an Inf":
        x[:, 5] = float("inf")
    elif kind == "nine Inf":
        x[:, 100:1000:100] = float("inf")
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


@pytest.mark.parametrize("gs", [2560, 4096 - 128, 6144, 8192, 11008])
@pytest.mark.parametrize("kind", ["silu", "quarters", "eighths", "clipped", "equals", "an Inf", "nine Inf"])
def test_kinds_of_data(kind, gs):
    check_line(kind, gs, 128, 8)


@pytest.mark.parametrize("gs,k,gq", [(2056, 1, 2056), (2560, 8, 512), (3080, 5, 8), (4088, 8, 4088), (4104, 2, 8), (6144, 7, 64), (8192, 8, 128),
                                     (8200, 3, 8200), (11264, 8, 256)])
def test_octets_that_the_list_cannot_hold(gs, k, gq):
    """More than the 16 octets of the list at the bound: 15 to 18 octets of equals beside fewer than k, k and more larger ones in one
    octet and in many, equals that begin in the octets of the larger ones, coarse values of many levels, rows of zeros
    with fewer than k others, and the tensor's last group of one octet."""
    for dtype, bits, asym in ((torch.bfloat16, 4, 0), (torch.float16, 8, 1)):
        g = torch.Generator().manual_seed(gs + k)
        x = torch.randn(GROUPS * gs + 8, generator=g)
        rows = x[:GROUPS * gs].view(GROUPS, gs)
        r = 0
        for octets in (14, 15, 16, 17, 18, 40, gs // 8):
            for larger in (0, 1, k - 1, k, k + 1, 12):
                rows[r, 0:8 * octets:8] = -9.0               # one in each of the first octets
                rows[r, gs - 8 * larger:gs:8] = 11.0          # the larger ones, one to an octet at the end
                r += 1
                rows[r, 3:8 * octets:8] = 9.0
                rows[r, 8:8 + min(larger, 8)] = 11.0          # .. or together in the second octet, equals among them
                rows[r, 8:8 + larger // 2] = 12.0
                r += 1
        for step in (0.25, 0.5, 1.0, 4.0):
            rows[r:r + 40] = (rows[r:r + 40] / step).round() * step
            r += 40
        for n in range(k + 2):                                # n values that are not zero
            rows[r] = 0.0
            rows[r, torch.randperm(gs, generator=g)[:n]] = torch.randn(n, generator=g)
            r += 1
        for n in (k - 1, k, k + 1):                           # so many that are not finite, beside many equals
            rows[r, ::16] = 9.0
            rows[r, gs // 3:gs // 3 + n] = float("nan")
            r += 1
            rows[r, ::16] = 9.0
            rows[r, 5:5 + 64 * n:64] = float("-inf")
            r += 1
        assert r < GROUPS
        x[GROUPS * gs:] = 2.0
        print(f"[list] gs={gs} k={k} gq={gq} {dtype} int{bits} asym={asym}", flush=True)
        run_parity(x.to(dtype), dict(bits=bits, quant_group=gq, asym=asym, outlier_mode="topk", stat_group=gs, thresh=0.0, topk=k))
