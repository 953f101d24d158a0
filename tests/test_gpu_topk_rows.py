"""TOPK over a tile or a segment that is one group: the threshold by halving, where it can go wrong - several of the k in one octet,
equals at the k-th place in one octet, one wavefront or all over the segment, more octets in question than a wavefront
looks at (a constant segment), values that are not finite, fewer elements than k."""
import pytest
import torch

from helpers import run_parity

pytestmark = pytest.mark.gpu


def rows(kind, gs, g):
    x = torch.randn(gs, generator=g) * 0.1
    if kind == "one_octet":
        x[16:24] = torch.tensor([5.0, 4.0, -6.0, 7.0, 3.0, 8.0, -9.0, 2.0])
    elif kind == "equals_in_an_octet":
        x[gs - 8:] = 3.0
        x[5] = 4.0
    elif kind == "equals_all_over":
        x[torch.randperm(gs, generator=g)[:40]] = -2.0
        x[7] = 2.5
    elif kind == "constant":
        x[:] = 1.25
    elif kind == "zeros":
        x[:] = 0.0
        x[gs // 2] = 1e-3
    elif kind in ("9", "16", "17"):  # octets with equals, the last of them with two
        at = 8 * torch.randperm(gs // 8, generator=g)[:int(kind)]
        x[at] = 2.0
        x[at[-1] + 5] = 2.0
    elif kind == "sixty_four_octets":
        x[8 * torch.randperm(gs // 8, generator=g)[:64]] = 2.0
    elif kind == "sixty_five_octets":
        x[8 * torch.randperm(gs // 8, generator=g)[:65]] = 2.0
    elif kind == "not_finite":
        x[::gs // 5] = float("inf")
        x[3] = float("nan")
    return x


@pytest.mark.parametrize("k", [1, 2, 3, 5, 8, 9])
@pytest.mark.parametrize("gs", [2048, 4096, 5160, 8192, 11008, 16384])
def test_threshold_of_a_row(k, gs):
    g = torch.Generator().manual_seed(k * gs)
    kinds = ["random", "one_octet", "equals_in_an_octet", "equals_all_over", "constant", "zeros", "sixty_four_octets",
             "sixty_five_octets", "not_finite", "9", "16", "17", "random"]
    for dtype, end in ((torch.bfloat16, 5), (torch.float16, 1001)):
        x = torch.cat([rows(kind, gs, g) for kind in kinds] + [rows("equals_all_over", gs, g)[:end]]).to(dtype)
        print(f"[topk row] k={k} gs={gs} {dtype}", flush=True)
        run_parity(x, dict(bits=4, quant_group=gs if gs == 5160 else 128, asym=0, outlier_mode="topk", stat_group=gs, thresh=0.0, topk=k))
