"""Long tensors are restored in smaller pieces (2 or 4 rows of a wavefront): both sides of the lines, compared with the pieces of 2048 elements
that batch calls keep, and with the compressed values where a batch goes the same way."""
import pytest
import torch

import paper_2508_00806_amd as adacc
from helpers import adacc_method

pytestmark = pytest.mark.gpu


def _method(mode, bits, asym, gq, gs, thresh, k, n):
    return adacc_method(dict(bits=bits, quant_group=gq, asym=asym, outlier_mode=mode, stat_group=gs, thresh=thresh, topk=k), n // 4)


def _tensor(n):
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(n, generator=g, device="cuda").to(torch.bfloat16)
    for first in (0, 2048 * 700, n - 70000):  # tiles full of outliers, chunks with several, tiles with none
        x[first:first + 3000] *= 30.0
        x[first + 4096:first + 4096 + 2048] *= 0.01
    x[5::4099] = 77.0
    x[6::8198] = -55.0
    x[-1] = float("inf")
    return x


def _both(m, x, f32):
    lay = adacc.layout_of(m, x.numel())
    blob = torch.zeros(lay.total_bytes, dtype=torch.uint8, device="cuda")
    adacc.compress(m, x, blob, adacc.alloc_workspace(max(adacc.workspace_bytes(m, x.numel()), 512)))
    one, many = (torch.zeros(x.numel(), dtype=torch.float32 if f32 else x.dtype, device="cuda") for _ in range(2))
    adacc.decompress(m, blob, one)
    ws = adacc.alloc_workspace(adacc.batch_workspace_bytes([m], [x.numel()]))
    adacc.decompress_batch([m], [blob], [many], ws)
    return blob, one, many


CASES = [("none", 8, 0, 64, 0, 0.0, 0), ("none", 4, 1, 128, 0, 0.0, 0), ("std", 8, 0, 64, 512, 3.0, 0), ("std", 4, 0, 256, 4096, 3.5, 0),
         ("abs", 8, 1, 4096, 0, 3.0, 0), ("topk", 4, 0, 128, 4096, 0.0, 5)]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("n,f32", [((1 << 25) - 8, True), ((1 << 25) + 8200, True), ((1 << 25) + 777, True), ((1 << 26) + 1031, False),
                                   ((1 << 28) + 2059, False)])
def test_small_pieces_restore_what_the_others_do(case, n, f32):
    mode, bits, asym, gq, gs, thresh, k = case
    x = _tensor(n)
    print(f"[pieces] {case} n={n} f32={f32}", flush=True)
    _, one, many = _both(_method(mode, bits, asym, gq, gs, thresh, k, n), x, f32)
    assert torch.equal(one.view(torch.int32 if f32 else torch.int16), many.view(torch.int32 if f32 else torch.int16))


@pytest.mark.parametrize("case", [("none", 8, 0, 40, 0, 0.0, 0), ("std", 8, 0, 8200, 8200, 3.0, 0), ("topk", 4, 1, 96, 11040, 0.0, 5)])
def test_groups_of_any_size(case):
    """The fallback methods in binary32: rounded, what they are in 16 bits."""
    mode, bits, asym, gq, gs, thresh, k = case
    n = (1 << 25) + 4107
    m, x = _method(mode, bits, asym, gq, gs, thresh, k, n), _tensor(n)
    blob, wide, _ = _both(m, x, True)
    narrow = torch.zeros_like(x)
    adacc.decompress(m, blob, narrow)
    assert torch.equal(wide.to(torch.bfloat16).view(torch.int16), narrow.view(torch.int16))


def _binary16(mode, bits, asym, gq, gs, thresh, k, n):
    m = adacc_method(dict(bits=bits, quant_group=gq, asym=asym, outlier_mode=mode, stat_group=gs, thresh=thresh, topk=k), n // 4, fmt=1)
    return m, _tensor(n).to(torch.float16)


@pytest.mark.parametrize("case,n,f32", [(c, n, f32) for c in CASES for n, f32 in (((1 << 25) + 777, True), ((1 << 26) + 1031, False))] +
                         [(c, (1 << 28) + 2059, False) for c in CASES[2:4]])
def test_small_pieces_in_binary16(case, n, f32):
    m, x = _binary16(*case, n)
    print(f"[pieces] binary16 {case} n={n} f32={f32}", flush=True)
    _, one, many = _both(m, x, f32)
    assert torch.equal(one.view(torch.int32 if f32 else torch.int16), many.view(torch.int32 if f32 else torch.int16))


@pytest.mark.parametrize("case", [("none", 8, 0, 40, 0, 0.0, 0), ("std", 8, 0, 8200, 8200, 3.0, 0), ("topk", 4, 1, 96, 11040, 0.0, 5)])
def test_groups_of_any_size_in_binary16(case):
    n = (1 << 25) + 4107
    m, x = _binary16(*case, n)
    blob, wide, _ = _both(m, x, True)
    narrow = torch.zeros_like(x)
    adacc.decompress(m, blob, narrow)
    assert torch.equal(wide.to(torch.float16).view(torch.int16), narrow.view(torch.int16))
