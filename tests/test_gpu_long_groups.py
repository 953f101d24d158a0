"""Groups of more than 2048 elements, enough of them that a wavefront takes each: at the edges of the numbers of rows that the kernels
exist for, with the tensor's last group short or one octet long, and with groups of every difficult kind among the others.
A tensor whose last octet is ragged, one group too few and quantisation groups that do not line up with a row take the workgroups' kernels;
all of it is compared with the oracle bit for bit."""
import pytest
import torch

from helpers import run_parity

pytestmark = pytest.mark.gpu

GROUPS = 3072  # from here on a wavefront per group


def tensor(gs, n, end, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.nn.functional.silu(torch.randn(n * gs + end, generator=g) * 1.5)
    rows = x[:n * gs].view(n, gs)
    rows[1] = 1.25                     # a constant
    rows[2] = 0.0
    rows[2, gs - 1] = -3.0
    rows[3, 5] = float("inf")
    rows[4, gs - 2] = float("nan")
    rows[5, ::7] = float("-inf")       # more than any k
    rows[6, 8:16] = 40.0               # an octet of outliers
    rows[7, 512:612] = -30.0           # more than a slot holds
    rows[8] *= 1e-20 if dtype == torch.bfloat16 else 1e-6
    rows[9] *= 1e18 if dtype == torch.bfloat16 else 1e4
    rows[10] = torch.where(rows[10] > 1.0, 4.0, 2.0)
    rows[11] = -rows[11].abs()
    return x.to(dtype)


@pytest.mark.parametrize("gs,end,mode,par,gq", [
    (2056, 0, "std", 4.0, 2056), (2056, 1000, "topk", 4, 2056), (2056, 8, "abs", 3.0, 2056), (2056, 0, "none", 0, 2056),
    (2560, 0, "topk", 8, 512), (3072, 0, "topk", 9, 8), (2304, 2296, "std", 3.0, 128), (3072, 2048, "none", 0, 3072), (3080, 0, "none", 0, 3080),
    (4088, 0, "std", 4.0, 4088), (4104, 0, "std", 4.0, 8), (4104, 8, "abs", 3.0, 4104), (6144, 8, "std", 4.0, 512), (6152, 4096, "std", 5.0, 6152), (8192, 0, "std", 4.0, 64),
    (8200, 0, "std", 4.0, 8200), (11264, 11256, "std", 4.0, 256), (11272, 0, "std", 4.0, 11272),
    (2056, 1003, "std", 4.0, 2056), (2400, 0, "std", 4.0, 96)])
def test_groups_of_many_rows(gs, end, mode, par, gq):
    for dtype, bits, asym, n in ((torch.bfloat16, 8, 0, GROUPS), (torch.float16, 4, 1, GROUPS), (torch.bfloat16, 4, 0, GROUPS - 1)):
        print(f"[long groups] gs={gs} n={n} + {end} {mode} {par} gq={gq} {dtype} int{bits} asym={asym}", flush=True)
        x = tensor(gs, n, end, dtype, gs + end)
        run_parity(x, dict(bits=bits, quant_group=gq, asym=asym, outlier_mode=mode, stat_group=gs if mode in ("std", "topk") else 0,
                           thresh=float(par) if mode in ("std", "abs") else 0.0, topk=par if mode == "topk" else 0))


@pytest.mark.parametrize("gs,end,k,gq", [
    (4104, 0, 4, 4104), (6144, 8, 8, 512), (6152, 4096, 1, 8), (8192, 0, 2, 64), (8200, 2000, 8, 8200), (11008, 0, 8, 128),
    (11264, 11256, 5, 256), (11264, 0, 3, 11264), (11272, 0, 8, 11272), (8192, 0, 9, 128), (11008, 5000, 8, 344)])
def test_the_largest_of_groups_of_many_rows(gs, end, k, gq):
    """Up to 8 of the largest by a wavefront, over 9 to 22 of its rows: equals at the k-th place, few and many, in one octet, in the last
    octet of the group, beside and beyond values that are not finite; 23 rows, 9 of the largest and quantisation groups that do
    not line up with a row by the workgroups."""
    for dtype, bits, asym, n in ((torch.bfloat16, 4, 0, GROUPS), (torch.float16, 8, 1, GROUPS)):
        print(f"[long groups, topk] gs={gs} n={n} + {end} k={k} gq={gq} {dtype} int{bits} asym={asym}", flush=True)
        x = tensor(gs, n, end, dtype, gs + k)
        rows = x[:n * gs].view(n, gs)
        rows[12, ::64] = 9.0               # equals by the dozen, none larger
        rows[13, 3::96] = -9.0             # the same below a few that are larger
        rows[13, 40:40 + k // 2] = 11.0
        rows[14, ::50] = 9.0               # .. beside values that are not finite
        rows[14, 17] = float("nan")
        rows[15, 100:100 + 8 * k:8] = float("inf")   # exactly k of them
        rows[16, gs - 8:] = 9.0            # the last octet, all of it equal
        rows[17, 1024:1040] = 9.0          # two octets of equals
        rows[18] = 0.0                     # nothing at all
        rows[19] = 0.0
        rows[19, gs // 2:gs // 2 + 3] = 1.0
        rows[20] = torch.tensor([1.0, -1.0, 0.5, 2.0]).repeat(gs // 4 + 1)[:gs].to(dtype)
        run_parity(x, dict(bits=bits, quant_group=gq, asym=asym, outlier_mode="topk", stat_group=gs, thresh=0.0, topk=k))
