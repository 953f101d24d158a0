"""Batches of few and of many short tensors: tables around the sizes of their uploads, tensors of very unequal length in one launch.
Every blob and every restored tensor is compared with what the single calls make of it."""
import pytest
import torch

import paper_2508_00806_amd as adacc
from helpers import adacc_method

pytestmark = pytest.mark.gpu

METHODS = [dict(bits=8, quant_group=64, asym=0, outlier_mode="none", stat_group=0, thresh=0.0, topk=0),
           dict(bits=4, quant_group=128, asym=0, outlier_mode="topk", stat_group=4096, thresh=0.0, topk=4),
           dict(bits=8, quant_group=64, asym=1, outlier_mode="std", stat_group=64, thresh=2.5, topk=0),
           dict(bits=4, quant_group=128, asym=0, outlier_mode="std", stat_group=512, thresh=2.5, topk=0)]


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 9, 17, 18, 35])
@pytest.mark.parametrize("f32", [False, True])
def test_short_and_long_tensors_in_one_launch(n, f32):
    g = torch.Generator().manual_seed(n)
    numels = [4096 * (1 + (37 * i) % 61) - (0 if i % 3 else 24 * (i % 2)) for i in range(n)]
    numels[-1] = 4096 * 300  # together beyond the line for n >= 14 or so
    methods, xs = [], []
    for i, numel in enumerate(numels):
        methods.append(adacc_method(METHODS[i % 4], numel // 8 + 64))
        xs.append(torch.randn(numel, generator=g).to(torch.bfloat16).cuda())
    lays = [adacc.layout_of(m, x.numel()) for m, x in zip(methods, xs)]

    def made():
        blobs = [torch.zeros(lay.total_bytes, dtype=torch.uint8, device="cuda") for lay in lays]
        outs = [torch.zeros(x.shape, dtype=torch.float32 if f32 else x.dtype, device="cuda") for x in xs]
        return blobs, outs
    one, many = made(), made()
    for m, x, b, o in zip(methods, xs, *one):
        adacc.compress(m, x, b, adacc.alloc_workspace(adacc.workspace_bytes(m, x.numel())))
        adacc.decompress(m, b, o)
    ws = adacc.alloc_workspace(adacc.batch_workspace_bytes(methods, numels))
    adacc.compress_batch(methods, xs, many[0], ws)
    adacc.decompress_batch(methods, many[0], many[1], ws)
    for i, (m, lay) in enumerate(zip(methods, lays)):
        for name, section in adacc.blob_sections(one[0][i], lay, m, numels[i]).items():
            assert torch.equal(section, adacc.blob_sections(many[0][i], lay, m, numels[i])[name]), (i, name)
        assert torch.equal(one[1][i], many[1][i]), i
