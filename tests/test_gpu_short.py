"""Short tensors whose outliers are found, ordered and stored in one launch: against the oracle, against the two launches that a
workspace without the room for it takes, and with the wavefronts counting for each other."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2508_00806_amd as adacc
import test_gpu_placement
import test_gpu_ragged
from helpers import adacc_method, run_parity

pytestmark = pytest.mark.gpu

# (quantisation group, statistics group, mode, threshold, topk, tile): the encoder by rows, the general one over 4 and 8 rows, TOPK of every kind
METHODS = [(64, 64, "std", 3.0, 0, 2048), (128, 512, "std", 2.5, 0, 2048), (256, 4096, "std", 2.5, 0, 4096), (512, 0, "abs", 1.5, 0, 2048),
           (4096, 0, "abs", 2.0, 0, 4096), (64, 1024, "topk", 0.0, 4, 2048), (128, 128, "topk", 0.0, 1, 2048),
           (128, 2048, "topk", 0.0, 5, 2048), (128, 4096, "topk", 0.0, 9, 4096), (4096, 4096, "topk", 0.0, 3, 4096)]


def _case(gq, gs, mode, thresh, k, bits, asym):
    return dict(bits=bits, quant_group=gq, asym=asym, outlier_mode=mode, stat_group=gs, thresh=thresh, topk=k)


def _values(n, tile, g, dtype):
    x = torch.randn(n, generator=g).to(dtype)
    for t in (0, 4, 5):  # tiles with more than a record holds, and one with values that are not finite
        x[t * tile:t * tile + 90] *= 20.0
    x[-3:] = float("nan")
    return x


@pytest.mark.parametrize("tiles,rest", [(0, 40), (1, 0), (3, 0), (4, 0), (5, 61), (63, 30), (64, 0), (257, 30), (1023, 0)])
@pytest.mark.parametrize("method", METHODS)
def test_against_the_oracle(method, tiles, rest):
    gq, gs, mode, thresh, k, tile = method
    if tiles > 300 and tile == 4096:
        tiles //= 2
    for bits, asym, dtype in ((8, 0, torch.bfloat16), (4, 1, torch.float16)):
        x = _values(tiles * tile + rest, tile, torch.Generator().manual_seed(tiles + gq), dtype)
        print(f"[short] {method} tiles={tiles} rest={rest} bits={bits}", flush=True)
        run_parity(x, _case(gq, gs, mode, thresh, k, bits, asym))


@pytest.mark.parametrize("tiles,rest", [(1, 0), (5, 61), (63, 30), (64, 0), (257, 30)])
@pytest.mark.parametrize("method", METHODS)
def test_two_launches_against_the_oracle(method, tiles, rest, monkeypatch):
    """The same tensors with workspaces that have no room for the words."""
    monkeypatch.setattr(adacc, "SHORT_BYTES", 0)
    test_against_the_oracle(method, tiles, rest)


def _compressed(m, x, ws):
    lay = adacc.layout_of(m, x.numel())
    blob = torch.zeros(lay.total_bytes, dtype=torch.uint8, device="cuda")
    adacc.compress(m, x, blob, ws)
    return blob


@pytest.mark.parametrize("tiles", [1280 * 4, 1280 * 4 + 1, 1792 * 4, 1792 * 4 + 1, 2560 * 4, 2560 * 4 + 1])
def test_the_same_as_in_two_launches(tiles):
    """Both sides of the lines in the number of workgroups; one workspace for all calls, with calls that need all of it between."""
    for gq, gs in ((64, 64), (64, 512)):
        n = tiles * 2048 + (40 if tiles > 1792 * 4 + 1 else 0)
        x = _values(n, 2048, torch.Generator().manual_seed(tiles), torch.bfloat16).cuda()
        m = adacc_method(_case(gq, gs, "std", 3.0, 0, 8, 0), n // 8)
        need = adacc.workspace_bytes(m, n)
        exact = adacc.Workspace(torch.empty(need, dtype=torch.uint8, device="cuda"))  # no room: two launches
        room = adacc.alloc_workspace(need)
        want = _compressed(m, x, exact)
        assert torch.equal(_compressed(m, x, room), want)
        part = x[:2048 * 9 + 64 * 5]
        mp = adacc_method(_case(gq, gs, "std", 3.0, 0, 8, 0), part.numel())
        short = _compressed(mp, part, room)
        assert room.c.reserved == 1
        assert torch.equal(_compressed(mp, part, exact), short)
        longer = adacc.Workspace(torch.empty(need + 256, dtype=torch.uint8, device="cuda"))
        assert torch.equal(_compressed(mp, part, longer), short)
        assert longer.c.reserved == 1
        assert torch.equal(_compressed(m, x, longer), want)  # needs the words' place
        assert longer.c.reserved == 0
        assert torch.equal(_compressed(mp, part, longer), short)
        for _ in range(3):  # other inputs through the same words
            x = x.flip(0)
            assert torch.equal(_compressed(m, x, room), _compressed(m, x, exact))


# (method, tiles, elements behind them, one launch): both sides of every line, and what has no short way
ROUTES = [(METHODS[0], 1280 * 4, 0, True), (METHODS[0], 1280 * 4 + 1, 0, False), (METHODS[3], 1280 * 4, 40, True), (METHODS[3], 1280 * 4 + 1, 40, False),
          (METHODS[1], 1792 * 4, 0, True), (METHODS[1], 1792 * 4 + 1, 0, False), (METHODS[1], 1792 * 4 + 1, 40, True),
          (METHODS[1], 2560 * 4, 40, True), (METHODS[1], 2560 * 4 + 1, 40, False), (METHODS[4], 1792 * 4, 0, True), (METHODS[4], 1792 * 4 + 1, 0, False),
          (METHODS[5], 256 * 4, 0, True), (METHODS[5], 256 * 4 + 1, 0, False), (METHODS[8], 256 * 4, 9, True), (METHODS[8], 256 * 4 + 1, 9, False),
          ((128, 128, "topk", 0.0, 4, 2048), 20, 0, True), ((128, 128, "topk", 0.0, 5, 2048), 20, 0, False), ((40, 40, "std", 3.0, 0, 4080), 20, 0, False),
          (METHODS[1], 1, 0, True), (METHODS[1], 0, 40, True)]


def _words(ws, workgroups):
    off = (ws.c.bytes - adacc.SHORT_BYTES) // 256 * 256
    return ws.buffer[off:off + 8 * workgroups].view(torch.int64)


@pytest.mark.parametrize("method,tiles,rest,one", ROUTES)
def test_which_calls_take_one_launch(method, tiles, rest, one):
    """A call in one launch leaves its number and a count in every workgroup's word, another one leaves them alone."""
    gq, gs, mode, thresh, k, tile = method
    n = tiles * tile + rest
    m = adacc_method(_case(gq, gs, mode, thresh, k, 8, 0), n // 8)
    x = torch.randn(n, generator=torch.Generator().manual_seed(n)).to(torch.bfloat16).cuda()
    ws = adacc.alloc_workspace(adacc.workspace_bytes(m, n))
    words = _words(ws, max((tiles + 3) // 4, 1))
    print(f"[route] {method} tiles={tiles} rest={rest}", flush=True)
    found = adacc.read_status(_compressed(m, x, ws), adacc.layout_of(m, n))[0]
    seen = words.cpu()
    if not one or tiles == 0:
        assert not seen.any()
        return
    assert bool((seen < 0).all()) and len(set((seen >> 16).tolist())) == 1  # (the top bit is part of a word)
    counts = int((seen & 0xFFFF).sum())
    assert counts == found if rest == 0 else counts <= found


def test_a_captured_call_takes_two_launches():
    n = 2048 * 70
    m = adacc_method(_case(64, 512, "std", 2.5, 0, 8, 0), n // 8)
    x = _values(n, 2048, torch.Generator().manual_seed(5), torch.bfloat16).cuda()
    ws = adacc.alloc_workspace(adacc.workspace_bytes(m, n))
    blob = torch.zeros(adacc.layout_of(m, n).total_bytes, dtype=torch.uint8, device="cuda")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        adacc.compress(m, x, blob, ws)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert not _words(ws, 18).any()
        assert torch.equal(blob, _compressed(m, x, adacc.alloc_workspace(adacc.workspace_bytes(m, n))))


# what these compare went over to one launch with the workspaces' room: the same once more without it
@pytest.mark.parametrize("fmt", [0, 1])
@pytest.mark.parametrize("mode", ["abs", "std", "topk"])
def test_short_last_groups_in_two_launches(mode, fmt, monkeypatch):
    monkeypatch.setattr(adacc, "SHORT_BYTES", 0)
    test_gpu_ragged.test_short_last_groups(mode, fmt)


@pytest.mark.parametrize("rest", [1, 8, 1999, 2048, 2049, 4095])
@pytest.mark.parametrize("mode", ["abs", "std", "topk"])
def test_the_end_of_a_tensor_in_two_launches(mode, rest, monkeypatch):
    monkeypatch.setattr(adacc, "SHORT_BYTES", 0)
    test_gpu_placement.test_the_end_of_a_tensor_that_its_groups_do_not_divide(mode, rest)


@pytest.mark.parametrize("shape", test_gpu_placement.SHAPES[:4])
def test_slots_at_their_limit_in_two_launches(shape, monkeypatch):
    monkeypatch.setattr(adacc, "SHORT_BYTES", 0)
    test_gpu_placement.test_slots_at_their_limit(*shape)


def test_two_structs_of_one_workspace():
    """Launches through copies of the host struct, whose counters repeat, on one buffer."""
    n = 2048 * 70
    m = adacc_method(_case(64, 512, "std", 2.5, 0, 8, 0), n // 8)
    xs = [_values(n, 2048, torch.Generator().manual_seed(s), torch.bfloat16).cuda() for s in (1, 2)]
    want = [_compressed(m, x, adacc.alloc_workspace(adacc.workspace_bytes(m, n))) for x in xs]
    ws = adacc.alloc_workspace(adacc.workspace_bytes(m, n))
    other = adacc.Workspace(ws.buffer)
    for _ in range(4):
        for x, w, b in zip(xs, (ws, other), want):
            assert torch.equal(_compressed(m, x, w), b)


def _overwritten_words():
    """Two structs of one buffer: before every short call through the one, a long call through the other leaves in the words' place slots whose
    first record is the element whose number is that of the short call in this process."""
    long, short = 2048 * 9000, 2048 * 7000
    ml, ms = (adacc_method(_case(1024, 0, "abs", 2.5, 0, 8, 0), n // 8) for n in (long, short))
    buffer = torch.empty(adacc.workspace_bytes(ml, long), dtype=torch.uint8, device="cuda")
    one, other = adacc.Workspace(buffer), adacc.Workspace(buffer)
    exact = adacc.Workspace(torch.empty(adacc.workspace_bytes(ms, short), dtype=torch.uint8, device="cuda"))
    x = (torch.rand(long, generator=torch.Generator().manual_seed(1)) - 0.5).to(torch.bfloat16).cuda()
    y = torch.randn(short, generator=torch.Generator().manual_seed(2)).to(torch.bfloat16).cuda()
    want = _compressed(ms, y, exact)
    for launch in range(1, 9):
        z = x.clone()
        z[launch::2048] = 3.0
        _compressed(ml, z, one)
        assert torch.equal(_compressed(ms, y, other), want), launch


def _in_a_process_of_its_own(code, **env):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = "import sys; sys.path[:0] = ['tests', '.']; import torch; import test_gpu_short as t\n" + code + "\nprint('all done')"
    r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, **env), cwd=root, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and "all done" in r.stdout, r.stderr[-2000:]


def test_words_that_another_struct_has_overwritten():
    _in_a_process_of_its_own("t._overwritten_words()")


def test_two_streams_at_a_time():
    """Launches that wait for their own workgroups side by side, each stream with a workspace of its own."""
    n = 2048 * 4 * 2000 + 24
    m = adacc_method(_case(64, 512, "std", 2.5, 0, 8, 0), n // 8)
    lay = adacc.layout_of(m, n)
    xs = [_values(n, 2048, torch.Generator().manual_seed(s), torch.bfloat16).cuda() for s in (1, 2)]
    spaces = [adacc.alloc_workspace(adacc.workspace_bytes(m, n)) for _ in xs]
    want = [_compressed(m, x, w) for x, w in zip(xs, spaces)]
    blobs = [torch.zeros(lay.total_bytes, dtype=torch.uint8, device="cuda") for _ in xs]
    streams = [torch.cuda.Stream() for _ in xs]
    torch.cuda.synchronize()
    for _ in range(20):
        for x, w, b, s in zip(xs, spaces, blobs, streams):
            adacc.compress(m, x, b, w, stream=s)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, blobs))


def test_wavefronts_that_count_for_others():
    """One look at the words, then the tiles that are missing are counted by the wavefront itself."""
    code = ("import sys; sys.path[:0] = ['tests', '.']; import torch; import test_gpu_short as t\n"
            "for m in t.METHODS:\n    t.test_against_the_oracle(m, 257, 30)\nprint('counted')")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, ADACC_SHORT_POLLS="1"), cwd=root, capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and "counted" in r.stdout, r.stderr[-2000:]


def test_wavefronts_that_count_for_others_over_many_words():
    """The same with more workgroups than a workgroup looks at together: every word once, what is missing counted by some and found by the rest."""
    _in_a_process_of_its_own("for m in t.METHODS[:5]: t.test_against_the_oracle(m, 1301 if m[5] == 2048 else 2605, 30)", ADACC_SHORT_POLLS="1")


def test_beside_kernels_that_hold_the_device():
    """Launches on one stream while long ones on another leave them some compute units at a time."""
    n = 2048 * 4 * 1700 + 24
    m = adacc_method(_case(64, 512, "std", 2.5, 0, 8, 0), n // 8)
    x = _values(n, 2048, torch.Generator().manual_seed(3), torch.bfloat16).cuda()
    ws = adacc.alloc_workspace(adacc.workspace_bytes(m, n))
    want = _compressed(m, x, ws)
    plain = adacc_method(_case(64, 0, "none", 0.0, 0, 8, 0), 0)
    y = torch.randn(1 << 27, device="cuda").to(torch.bfloat16)
    blob = torch.zeros(adacc.layout_of(plain, y.numel()).total_bytes, dtype=torch.uint8, device="cuda")
    blobs = [torch.zeros_like(want) for _ in range(12)]
    torch.cuda.synchronize()
    one, other = torch.cuda.Stream(), torch.cuda.Stream()
    for b in blobs:
        for _ in range(4):
            adacc.compress(plain, y, blob, stream=one)
        adacc.compress(m, x, b, ws, stream=other)
    torch.cuda.synchronize()
    assert all(torch.equal(b, want) for b in blobs)
