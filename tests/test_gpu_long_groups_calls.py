"""A wavefront per group of more than 2048 elements (3072 groups and more): with the divisor of the full range, with a stream that holds fewer
outliers than there are, and through a batch call; and batch calls in both formats for every class of kernel, with both
divisors, symmetric and asymmetric.  Bit for bit with the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_00806_amd as adacc
from helpers import adacc_method, bits_of, compare_blob_with_oracle, fmt_of, oracle_method, run_parity

pytestmark = pytest.mark.gpu

GROUPS = 3072  # from here on a wavefront per group


def method(mode, par, gs, gq, bits, asym):
    return dict(bits=bits, quant_group=gq, asym=asym, outlier_mode=mode, stat_group=gs if mode in ("std", "topk") else 0,
                thresh=float(par) if mode in ("std", "abs") else 0.0, topk=par if mode == "topk" else 0)


def tensor(n, gs, dtype):
    x = torch.nn.functional.silu(torch.randn(n, generator=torch.Generator().manual_seed(n)) * 1.5)
    rows = x[:n // gs * gs].view(-1, gs)
    rows[0] = 0.75
    rows[1, ::9] = -8.0
    rows[2, gs // 2] = float("nan")
    rows[-1, :] = (rows[-1] * 2).round() / 2
    return x.to(dtype)


@pytest.mark.parametrize("gs,gq,mode,par", [(2200, 2200, "std", 3.0), (2560, 128, "topk", 8), (3072, 3072, "none", 0), (6152, 6152, "abs", 3.0),
                                            (6656, 512, "topk", 3), (8192, 8192, "std", 4.0), (11008, 64, "std", 4.0), (11264, 256, "topk", 8)])
def test_divisor_of_the_full_range(gs, gq, mode, par):
    for dtype, bits, asym in ((torch.bfloat16, 4, 0), (torch.bfloat16, 8, 1), (torch.float16, 8, 0), (torch.float16, 4, 1)):
        print(f"[long, full range] gs={gs} gq={gq} {mode} {dtype} int{bits} asym={asym}", flush=True)
        run_parity(tensor(GROUPS * gs, gs, dtype), method(mode, par, gs, gq, bits, asym), rule=1)


@pytest.mark.parametrize("gs,mode,par", [(2560, "topk", 8), (8192, "topk", 5), (2560, "std", 3.0), (6656, "std", 3.0), (5120, "abs", 2.0)])
def test_a_stream_that_overflows(gs, mode, par):
    """Room for a third of the outliers, for all but one, and for none but one: what fits is there, the count is the whole count."""
    x = tensor(GROUPS * gs + 8, gs, torch.bfloat16)
    md = method(mode, par, gs, 128, 4, 0)
    n = oracle.compress(oracle_method(md, fmt=0), bits_of(x)).n_out
    for cap in (n // 3, n - 1, 1):
        print(f"[long, overflow] gs={gs} {mode} outliers={n} room={cap}", flush=True)
        run_parity(x, md, cap=cap)


# (elements, statistics group, quantisation group, mode, parameter); one of each class of batch kernels, and the long groups, which a batch
# call launches by themselves
CLASSES = [(2048 * 33 + 77, 64, 64, "std", 3.0), (2048 * 20, 512, 512, "topk", 3), (2048 * 40 + 512, 512, 64, "std", 3.0), (2048 * 25, 1024, 128, "topk", 4),
           (2048 * 30 + 1024, 1024, 1024, "abs", 2.5), (2048 * 18 + 3, 2048, 2048, "none", 0), (2048 * 21, 2048, 128, "topk", 2), (4096 * 13, 4096, 64, "std", 4.0),
           (4096 * 11, 4096, 4096, "topk", 4), (4096 * 9 + 100, 4096, 4096, "none", 0), (4096 * 17, 4096, 256, "topk", 8), (2200 * GROUPS, 2200, 2200, "std", 4.0),
           (2560 * GROUPS + 16, 2560, 512, "topk", 8)]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("bits,asym,rule", [(4, 0, 0), (8, 1, 0), (8, 0, 1), (4, 1, 1)])
def test_batches_of_every_class(dtype, bits, asym, rule):
    table = []
    for n, gs, gq, mode, par in CLASSES:
        x, md = tensor(n, gs, dtype), method(mode, par, gs, gq, bits, asym)
        oc = oracle.compress(oracle_method(md, rule, fmt_of(x)), bits_of(x))
        oc._full_idx = oc.out_idx.astype(np.int64)
        m = adacc_method(md, max(oc.n_out, 1) if mode != "none" else 0, rule, fmt_of(x))
        blob, L = adacc.alloc_blob(m, n)
        table.append((x.cuda(), m, blob, L, oc))
    srcs, methods, blobs, layouts, ocs = (list(c) for c in zip(*table))
    ws = adacc.alloc_workspace(adacc.batch_workspace_bytes(methods, [s.numel() for s in srcs]))
    print(f"[batch classes] {dtype} int{bits} asym={asym} rule={rule}: {len(methods)} tensors", flush=True)
    adacc.compress_batch(methods, srcs, blobs, ws)
    outs = [torch.empty_like(s) for s in srcs]
    adacc.decompress_batch(methods, blobs, outs, ws)
    torch.cuda.synchronize()
    for (n, gs, gq, mode, par), m, blob, L, oc, out in zip(CLASSES, methods, blobs, layouts, ocs, outs):
        print(f"[batch classes] gs={gs} gq={gq} {mode}", flush=True)
        compare_blob_with_oracle(blob, L, m, n, oc)
        want = oracle.decompress(oc)[1]
        nan = (want & 0x7FFF) > (0x7C00 if dtype == torch.float16 else 0x7F80)
        assert np.array_equal(bits_of(out)[~nan], want[~nan])
