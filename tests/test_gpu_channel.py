"""GPU parity for outlier channels by Z-score (Section 3.2, Eq. 1): libadacc's adacc_channel_*
calls (through the C ABI) against the CPU oracle.  Bar: the channel mask, list and values, packed
codes, scales and offsets bit-exact; decompressed binary32 bit-equal (hence within 1e-6), bf16 equal.
The oracle's channel sums are exact and the library's are binary32 partial sums in a fixed order, so
the helper also checks that no channel of a tested input has its Z within rounding reach of the
threshold (otherwise equal channel sets would prove nothing)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_00806_amd as adacc
import workloads
from helpers import bits_of, run_channel_parity

pytestmark = pytest.mark.gpu


def log(msg):
    print(msg, flush=True)


def planted(tokens, hidden, channels, seed, gain=50.0):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(tokens, hidden, generator=g)
    x[:, channels] *= gain
    return x.to(torch.bfloat16)


@pytest.mark.parametrize("bits,asym", [(4, 0), (8, 0), (4, 1), (8, 1)])
def test_activation_with_outlier_channels(bits, asym):
    """The workload of the paper's Fig. 3(a): a few channels carry the large magnitudes.  300 tokens:
    four whole chunks of 64 and a short one; every tile complete."""
    log(f"[channel] c2-shaped rows=300 bits={bits} asym={asym}")
    x = workloads.c2("cpu", rows=300)
    oc, _ = run_channel_parity(x, bits, 128, asym)
    assert oc.n_ch == 10
    log(f"[channel] n_ch={oc.n_ch} channels={list(oc.ch_idx)}")


def test_hidden_not_a_power_of_two_and_short_last_tile():
    log("[channel] hidden=11008 rows=37")
    x = planted(37, 11008, [0, 5000, 11007], seed=21)
    oc, _ = run_channel_parity(x, 8, 64, 1)
    assert set([0, 5000, 11007]) <= set(oc.ch_idx)


def test_narrow_matrix_with_neighbouring_outlier_channels():
    """A tile spans 51 tokens; channels 3 and 4 share an octet, 39 is the last one; threshold 2."""
    log("[channel] hidden=40 tokens=1000 z=2")
    x = planted(1000, 40, [3, 4, 17, 39], seed=22)
    oc, _ = run_channel_parity(x, 4, 8, 0, z=2.0)
    assert list(oc.ch_idx) == [3, 4, 17, 39]


@pytest.mark.parametrize("tokens", [203, 206, 5])
def test_strips_with_a_short_last_block_of_tokens(tokens):
    """Rows of 3 x 512 channels, groups inside 512 channels: the strip kernel (8 tokens per wavefront), with
    1 .. 7 tokens left for the last block; two outlier channels in one octet, the first and the last
    channel of a strip, and two channels kept because one of their values is not finite."""
    log(f"[channel] strips hidden=1536 tokens={tokens}")
    x = planted(tokens, 1536, [0, 511, 512, 700, 701, 1535], seed=24 + tokens)
    x[tokens // 2, 100] = float("inf")
    x[tokens - 1, 1400] = float("nan")
    for bits, gq, asym in ((4, 128, 0), (8, 512, 1), (4, 8, 1), (8, 64, 0)):
        oc, _ = run_channel_parity(x, bits, gq, asym)
        assert [int(i) for i in oc.ch_idx] == [0, 100, 511, 512, 700, 701, 1400, 1535]
    run_channel_parity(x.to(torch.float32).clamp(-6e4, 6e4).to(torch.float16), 4, 128, 0)


def test_widest_and_narrowest_matrices():
    """hidden = 65536 (the most the mode takes: 8 mask bytes per thread of the selection, 128 strips) with a
    short block of tokens, and hidden = 8 (one octet, one live lane in the statistics pass)."""
    log("[channel] hidden=65536 tokens=9")
    x = planted(9, 65536, [0, 7, 8, 32767, 40000, 65535], seed=31)
    oc, _ = run_channel_parity(x, 4, 512, 0)
    assert [int(i) for i in oc.ch_idx] == [0, 7, 8, 32767, 40000, 65535]
    log("[channel] hidden=8 tokens=100")
    x = planted(100, 8, [5], seed=32, gain=400.0)
    oc, _ = run_channel_parity(x, 8, 8, 1, z=2.0)
    assert [int(i) for i in oc.ch_idx] == [5]


def test_groups_of_a_whole_tile_and_the_other_scale_rule():
    log("[channel] hidden=4096 gq=2048")
    x = planted(70, 4096, [9, 10, 11, 12, 13, 14, 15, 16, 4000], seed=23)
    run_channel_parity(x, 8, 2048, 0, rule=1)
    run_channel_parity(x, 4, 1024, 1)


def test_degenerate_statistics():
    log("[channel] all channels alike / non-finite sums / one token")
    rng = np.random.default_rng(24)
    tokens, hidden = 64, 128
    mags = np.stack([rng.permutation(np.arange(1, tokens + 1)) for _ in range(hidden)], axis=1)
    x = torch.from_numpy((mags * rng.choice([-0.25, 0.25], size=(tokens, hidden))).astype(np.float32)).to(torch.bfloat16)
    oc, _ = run_channel_parity(x, 4, 64, 0)
    assert oc.n_ch == 0  # sigma = 0
    x = planted(130, 256, [7], seed=25)
    x[5, 100] = float("inf")
    x[77, 200] = float("nan")
    x[0, 201] = float("-inf")
    oc, _ = run_channel_parity(x, 8, 32, 1)
    assert list(oc.ch_idx) == [7, 100, 200, 201]
    run_channel_parity(planted(1, 2048, [11], seed=26), 8, 64, 0)  # a single token


def test_more_channels_than_the_blob_holds():
    log("[channel] capacity 1, two outlier channels")
    oc, st = run_channel_parity(planted(70, 64, [5, 40], seed=27), 8, 32, 0, cap=1)
    assert st[:2] == (2, 1)


def test_full_size_c2_shape():
    """[32768, 2048] in the launch configuration the bench times; every section compared."""
    log("[channel] full C2 shape")
    x = workloads.make("c2", "cpu")
    oc, _ = run_channel_parity(x, 4, 128, 0, cap=64)
    assert oc.n_ch == 10


def test_second_call_reuses_blob_and_workspace():
    """Nothing of an earlier call may leak into a later, smaller one."""
    log("[channel] reuse")
    tokens, hidden = 200, 512
    m = adacc.ChannelMethod(bits=8, quant_group=64, max_channels=8)
    blob, L = adacc.alloc_channel_blob(m, tokens, hidden)
    ws = adacc.alloc_channel_workspace(tokens, hidden)
    for seed, chans, t in ((28, [1, 2, 3, 300], tokens), (29, [450], 70)):
        x = planted(t, hidden, chans, seed)
        oc = oracle.channel_compress(oracle.Method(bits=8, quant_group=64), bits_of(x), t, hidden, 3.0, cap=8)
        adacc.channel_compress(m, x.cuda(), t, hidden, blob, ws)
        L2 = adacc.channel_layout_of(m, t, hidden)
        assert adacc.channel_read_status(blob, L2)[0] == oc.n_ch
        sec = {k: v.cpu().numpy() for k, v in adacc.channel_blob_sections(blob, L2, m, t, hidden).items()}
        assert np.array_equal(sec["codes"], oc.packed) and np.array_equal(sec["ch_idx"][:oc.n_ch], oc.ch_idx)
        assert np.array_equal(sec["ch_val"].view(np.uint16)[:t * oc.n_ch].reshape(t, oc.n_ch), oc.ch_val)


def test_repeat_launches_give_the_same_blob():
    """The library's sums have a fixed order: the same input gives the same bytes on every launch."""
    log("[channel] determinism")
    tokens, hidden = 1500, 1024
    x = workloads.c2("cpu", rows=tokens, hidden=hidden).cuda()
    m = adacc.ChannelMethod(bits=4, quant_group=128, max_channels=32)
    ws = adacc.alloc_channel_workspace(tokens, hidden)
    blobs = []
    for _ in range(3):
        blob, L = adacc.alloc_channel_blob(m, tokens, hidden)
        blob.zero_()
        adacc.channel_compress(m, x, tokens, hidden, blob, ws)
        torch.cuda.synchronize()
        n_ch = adacc.channel_read_status(blob, L)[0]
        sec = adacc.channel_blob_sections(blob, L, m, tokens, hidden)
        blobs.append((n_ch, {k: v.clone() for k, v in sec.items()}))
    for n_ch, sec in blobs[1:]:
        assert n_ch == blobs[0][0]
        for k in ("codes", "scales", "ch_mask", "ch_base"):
            assert torch.equal(sec[k], blobs[0][1][k]), k
        assert torch.equal(sec["ch_idx"][:n_ch], blobs[0][1]["ch_idx"][:n_ch])


@pytest.mark.parametrize("tokens,hidden,bits,asym", [(11, 1000, 4, 0), (3, 1416, 8, 1)])
def test_mask_of_a_matrix_that_is_no_multiple_of_a_tile(tokens, hidden, bits, asym):
    """Octets behind the end of the last tile are stored to a scrap area: not over the channel mask (bytes 64 .. 99 of
    it, channels 512 .. 799)."""
    x = torch.randn((tokens, hidden), generator=torch.Generator().manual_seed(hidden)).to(torch.bfloat16)
    for ch in (5, 520, 575, 640, 671, 770):
        x[:, ch] *= 60.0
    oc, _ = run_channel_parity(x, bits, 8, asym)
    assert oc.n_ch == 6
