"""Which stream waits for what when the hooks pack on one stream and unpack on another, without a GPU: streams, events
and library calls are stand-ins that write down the order in which they are used."""
import pytest
import torch

import paper_2508_00806_amd as adacc
import paper_2508_00806_amd.hooks as hooks


class Stream:
    def __init__(self, name, log):
        self.name, self.log, self.cuda_stream = name, log, id(self)

    def wait_event(self, event):
        self.log.append(("wait", self.name, event.after))

    def wait_stream(self, other):
        self.log.append(("wait", self.name, other.name))


@pytest.fixture
def world(monkeypatch):
    """log, a switch for the current stream, and a context whose library calls only write to the log."""
    log = []
    streams = {n: Stream(n, log) for n in ("a", "b")}  # (hashed and compared by identity)
    now = {"stream": streams["a"]}

    class Event:
        def __init__(self, enable_timing=False):
            self.after = None

        def record(self, stream=None):
            self.after = (stream or now["stream"]).name

        def synchronize(self):
            log.append(("host waits", self.after))

    def library(what):
        def call(*args, stream=None, **kw):
            log.append((what, stream.name))
            for t in args:
                if what in ("compress", "channel_compress") and isinstance(t, torch.Tensor) and t.dtype == torch.uint8:
                    t.zero_()  # the blob, status words among it
        return call

    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: now["stream"])
    monkeypatch.setattr(torch.cuda, "Event", Event)
    for name in ("compress", "decompress", "channel_compress", "channel_decompress", "mask_pack", "mask_unpack"):
        monkeypatch.setattr(hooks, name, library(name))
    monkeypatch.setattr(hooks._StatusPool, "take", lambda self: torch.zeros(4, dtype=torch.int32))
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda self, s: log.append(("keeps memory for", s.name)))
    monkeypatch.setattr(hooks.SavedActivationCompression, "_eligible", lambda self, t: True)
    return log, now, streams


def saved_on_a(method, world, tensor=None):
    log, now, streams = world
    ctx = hooks.SavedActivationCompression(lambda t: method, timing=False, pack_masks=False)
    t = torch.zeros(64, 1024, dtype=torch.bfloat16) if tensor is None else tensor
    saved = ctx._pack(t) if method is not None else ctx._pack_mask(t)
    del log[:]
    return ctx, saved


METHODS = {
    "groups": adacc.Method(bits=4, quant_group=128),
    "channels": adacc.ChannelMethod(bits=8, quant_group=64, z_thresh=3.0, max_channels=16),
    "mask": None,
}


@pytest.mark.parametrize("kind", sorted(METHODS))
def test_a_restoration_waits_for_the_stream_that_packed(kind, world):
    log, now, streams = world
    mask = torch.ones(4096, dtype=torch.bool) if kind == "mask" else None
    ctx, saved = saved_on_a(METHODS[kind], world, mask)
    now["stream"] = streams["b"]
    ctx._unpack(saved)
    restored = [i for i, e in enumerate(log) if e[0] in ("decompress", "channel_decompress", "mask_unpack")]
    assert len(restored) == 1 and log[restored[0]][1] == "b"
    assert ("wait", "b", "a") in log[:restored[0]], log
    assert ("keeps memory for", "b") in log  # graph and record may let go of the buffer while b still reads it
    if kind != "mask":  # and nobody sees the result before its status
        assert ("host waits", "a") in log[restored[0]:]


@pytest.mark.parametrize("kind", sorted(METHODS))
def test_one_stream_waits_for_nothing(kind, world):
    log, now, streams = world
    mask = torch.ones(4096, dtype=torch.bool) if kind == "mask" else None
    ctx, saved = saved_on_a(METHODS[kind], world, mask)
    ctx._unpack(saved)
    assert not [e for e in log if e[0] in ("wait", "keeps memory for")], log


@pytest.mark.parametrize("kind", ["groups", "channels"])
def test_streams_do_not_share_a_workspace(kind, world, monkeypatch):
    """Two compressions that may overlap need different workspaces; one stream keeps its own."""
    log, now, streams = world
    method = METHODS[kind] if kind == "channels" else adacc.Method(bits=4, quant_group=128, outlier_mode=adacc.OUTLIER_ABS, thresh=1.0,
                                                                   max_outliers=64)
    used = []

    class Workspace:
        def __init__(self, nbytes):
            self.c = type("c", (), {"bytes": nbytes})

    monkeypatch.setattr(hooks, "alloc_workspace", lambda nbytes, device=None: Workspace(nbytes))
    call = hooks.compress if kind == "groups" else hooks.channel_compress

    def note(*args, **kw):
        used.append(args[-1])
        call(*args[:-1], **kw)
        for t in args:  # the blob's status words
            if isinstance(t, torch.Tensor) and t.dtype == torch.uint8:
                t.zero_()
    monkeypatch.setattr(hooks, "compress" if kind == "groups" else "channel_compress", note)
    ctx = hooks.SavedActivationCompression(lambda t: method, timing=False, pack_masks=False)
    t = torch.zeros(64, 1024, dtype=torch.bfloat16)
    for name in "aabab":
        now["stream"] = streams[name]
        ctx._pack(t)
    assert used[0] is used[1] is used[3] and used[2] is used[4] and used[0] is not used[2]


def test_no_tensor_takes_the_room_behind_a_workspace(world, monkeypatch):
    """Tensors of growing size in one context: each finds a workspace that holds it in front of the last SHORT_BYTES, which compressions of
    short tensors in one launch use and lose once another call has reached into them."""
    made, used = [], []

    class Workspace:
        def __init__(self, nbytes):
            self.c = adacc.CWorkspace(256, (nbytes + 255) // 256 * 256 + adacc.SHORT_BYTES, 0, 1)
            made.append(self)
    monkeypatch.setattr(hooks, "alloc_workspace", lambda nbytes, device=None: Workspace(nbytes))

    def compress(m, t, blob, ws, stream=None):
        blob.zero_()
        used.append((ws, adacc.workspace_bytes(m, t.numel())))
    monkeypatch.setattr(hooks, "compress", compress)
    m = adacc.Method(bits=8, quant_group=64, outlier_mode=adacc.OUTLIER_STD, stat_group=64, thresh=4.0, max_outliers=64)
    ctx = hooks.SavedActivationCompression(lambda t: m, timing=False)
    for rows in (64, 8, 80, 96, 128, 100):  # 20480 bytes are 79 tiles
        ctx._pack(torch.zeros(rows, 2048, dtype=torch.bfloat16))
    assert all(ws.c.bytes - adacc.SHORT_BYTES >= need for ws, need in used) and len(used) == 6
    assert used[1][0] is used[0][0] and used[5][0] is used[4][0]  # kept where it is large enough
