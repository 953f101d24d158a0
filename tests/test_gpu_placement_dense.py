"""Tiles with more outliers than a slot of the workspace holds: the placement selects them again, sixteen wavefronts of a workgroup
sharing its 64 tiles (up to 16384 tiles; four beyond, and a window per wavefront from 32769 on).  Everything is compared bit by bit with the oracle."""
import pytest
import torch

import paper_2508_00806_amd as adacc
from helpers import run_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,tiles,rest,dtype", [(2048, 1, 0, torch.bfloat16), (2048, 15, 300, torch.float16), (2048, 63, 0, torch.bfloat16),
                                                  (2048, 65, 511, torch.bfloat16), (4096, 17, 4095, torch.bfloat16), (4096, 129, 0, torch.float16),
                                                  (2048, 1041, 77, torch.bfloat16), (2048, 16384, 5, torch.bfloat16), (2048, 16385, 5, torch.bfloat16),
                                                  (2048, 32769, 0, torch.bfloat16)])
@pytest.mark.parametrize("room", [0, adacc.SHORT_BYTES])  # none: two launches for every tensor
def test_dense_tiles(tile, tiles, rest, dtype, room, monkeypatch):
    monkeypatch.setattr(adacc, "SHORT_BYTES", room)
    n = tile * tiles + rest
    g = torch.Generator().manual_seed(n)
    x = (torch.rand(n, generator=g) - 0.5).to(dtype)
    few = tiles > 2000  # long: dense where workgroups, their wavefronts' shares and the windows begin and end
    for t in range(tiles):
        if few and t % 64 not in (0, 3, 4, 59, 60, 63) and t < tiles - 70:
            continue
        k = (64, 65, 200, 0, 66, tile)[t % 6] if not few else (65, 3, 70)[t % 3]
        if few and t > 300 and t < tiles - 300 and t % 7:
            continue
        at = t * tile + torch.randperm(tile, generator=g)[:k]
        x[at] = 3.0 + torch.rand(k, generator=g).to(dtype)
    x[-1] = float("-inf")
    print(f"[dense] tile={tile} tiles={tiles} rest={rest} {dtype}", flush=True)
    for gq, mode, thresh in ((64 if tile == 2048 else 4096, "abs", 1.0), (512 if tile == 2048 else 4096, "std", 2.0)):
        if few and mode == "std":
            continue
        oc, *_ = run_parity(x, dict(bits=8, quant_group=gq, asym=0, outlier_mode=mode, stat_group=gq if mode == "std" else 0,
                                    thresh=thresh, topk=0))
        assert oc.n_out > 0
