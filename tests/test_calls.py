"""The native marshalling of the binding's calls hands the library what the general way (ctypes) hands it, and leaves to that way what it
does not take.  The library's functions are stand-ins that write their arguments down; no GPU is involved."""
import ctypes
import os
import sysconfig
import warnings

import pytest
import torch

import paper_2508_00806_amd as adacc

U32, U64, VP, I = ctypes.c_uint32, ctypes.c_uint64, ctypes.c_void_p, ctypes.c_int
PM, PC, PW = ctypes.POINTER(adacc.CMethod), ctypes.POINTER(adacc.CChannelMethod), ctypes.POINTER(adacc.CWorkspace)
SIGNATURES = {"adacc_compress": (PM, VP, U64, VP, U64, PW, VP), "adacc_decompress": (PM, VP, U64, U64, VP, I, VP),
              "adacc_mask_pack": (VP, U64, VP, VP), "adacc_mask_unpack": (VP, U64, VP, VP),
              "adacc_channel_compress": (PC, VP, U64, U32, VP, U64, VP, U64, VP), "adacc_channel_decompress": (PC, VP, U64, U64, U32, VP, I, VP),
              "adacc_channelwise_compress": (U32, U32, U32, VP, U64, U32, VP, U64, VP, U64, VP),
              "adacc_channelwise_decompress": (U32, U32, VP, U64, U64, U32, VP, I, VP)}


def _plain(v):
    if isinstance(v, ctypes._Pointer):
        return tuple(getattr(v.contents, f) for f, _ in v.contents._fields_) if v else None
    return v or 0


@pytest.fixture
def world(monkeypatch):
    """(calls seen by the library, the switch between the two ways, what the library answers)"""
    seen, answer = [], [adacc.OK]
    real = adacc.lib()

    class Library:
        adacc_mask_packed_bytes, adacc_strerror = real.adacc_mask_packed_bytes, real.adacc_strerror

    for name, types in SIGNATURES.items():
        def stand_in(*args, name=name):
            seen.append((name, tuple(_plain(a) for a in args)))
            return answer[0]
        setattr(Library, name, ctypes.CFUNCTYPE(I, *types)(stand_in))
    monkeypatch.setattr(adacc, "_lib", Library)
    monkeypatch.setattr(adacc, "_calls", None)

    def general(on):
        if on:
            class Refuses:
                def __getattr__(self, name):
                    raise TypeError(name)
            monkeypatch.setattr(adacc, "_calls", Refuses())
        else:
            monkeypatch.setattr(adacc, "_calls", None)
    yield seen, general, answer
    monkeypatch.undo()
    adacc._calls = None  # bound anew to the real library


class Workspace(adacc.Workspace):
    def __init__(self):
        self.c = adacc.CWorkspace(4096, 512, 7, 1)
        self.address = ctypes.addressof(self.c)


def _workspace():
    w = Workspace()
    w.__class__ = adacc.Workspace
    return w


def _every_call():
    x, h = torch.zeros(3, 1000, dtype=torch.bfloat16), torch.zeros(3, 1000, dtype=torch.float16)
    blob, out, ws = torch.zeros(7777, dtype=torch.uint8), torch.zeros(3, 1000), torch.zeros(333, dtype=torch.int32)
    m = adacc.Method(bits=4, quant_group=128, asym=1, scale_rule=1, outlier_mode=adacc.OUTLIER_TOPK, stat_group=1024, thresh=0.1, topk=5, max_outliers=99)
    mh = adacc.Method(bits=8, quant_group=8, outlier_mode=adacc.OUTLIER_STD, stat_group=16, thresh=3, max_outliers=1, dtype=adacc.DTYPE_F16)
    c = adacc.ChannelMethod(bits=8, quant_group=64, z_thresh=2.5, max_channels=11)
    mask, w = torch.zeros(100, dtype=torch.bool), _workspace()
    yield lambda: adacc.compress(m, x, blob, w, stream=17)
    yield lambda: adacc.compress(m, x, blob, None, numel=2000, stream=0)
    yield lambda: adacc.compress(mh, 256, blob, stream=5, numel=8)
    yield lambda: adacc.decompress(m, blob, x, stream=3)
    yield lambda: adacc.decompress(m, blob, out, numel=17, stream=3)
    yield lambda: adacc.decompress(mh, blob, h, stream=1 << 40)
    yield lambda: adacc.decompress(mh, blob, x, stream=3)  # a TypeError: not the format of the method
    yield lambda: adacc.mask_pack(mask, blob, stream=4)
    yield lambda: adacc.mask_pack(mask, blob[:12], stream=4)  # too small
    yield lambda: adacc.mask_unpack(blob, mask, 9, stream=4)
    yield lambda: adacc.mask_unpack(blob, mask, 101, stream=4)
    yield lambda: adacc.channel_compress(c, x, 3, 1000, blob, ws, stream=6)
    yield lambda: adacc.channel_decompress(c, blob, 3, 1000, out, stream=6)
    yield lambda: adacc.channel_decompress(c, blob, 3, 1000, h, stream=6)
    yield lambda: adacc.channelwise_compress(4, h, 3, 1000, blob, ws, adacc.SCALE_FULLRANGE, stream=8)
    yield lambda: adacc.channelwise_decompress(8, blob, 3, 1000, h, stream=8)
    yield lambda: adacc.channelwise_decompress(8, blob, 3, 1000, blob, stream=8)
    yield lambda: adacc.compress(m, x, None, w, stream=17)  # no size to ask for
    yield lambda: adacc.compress(adacc.Method(bits=4.5), x, blob, stream=17)
    yield lambda: adacc.channel_compress(c, x, 3, 1000, blob, None, stream=6)

    class Own:  # a method of the caller's own
        dtype = adacc.DTYPE_BF16

        def c(self):
            return m.c()
    yield lambda: adacc.compress(Own(), x, blob, w, stream=17)
    yield lambda: adacc.decompress(Own(), blob, x, stream=17)


def _outcome(call):
    try:
        return call()
    except Exception as e:  # noqa: BLE001
        return type(e).__name__, getattr(e, "code", None)


@pytest.mark.parametrize("rc", [adacc.OK, adacc.EINVAL])
def test_both_ways_hand_over_the_same(world, rc):
    seen, general, answer = world
    answer[0] = rc
    for call in _every_call():
        general(True)
        want = _outcome(call), list(seen)
        del seen[:]
        general(False)
        assert (_outcome(call), list(seen)) == want
        del seen[:]


def test_what_is_not_marshalled_reaches_no_library_call(world):
    seen, general, _ = world
    x, blob = torch.zeros(64, dtype=torch.bfloat16), torch.zeros(4096, dtype=torch.uint8)
    native = adacc.calls()
    for args in ((adacc.Method(), x, blob, None, 64.0, 1), (adacc.Method(), x, blob, None, None), (adacc.Method(bits="8"), x, blob, None, None, 1)):
        with pytest.raises(TypeError):
            native.compress(*args)
    with pytest.raises(AttributeError):
        native.compress(object(), x, blob, None, None, 1)
    assert seen == []


def _broken(tmp_path, content):
    path = tmp_path / "_calls.so"
    if content is not None:
        path.write_bytes(content)
    return str(path)


@pytest.mark.parametrize("content", [None, b"not a library"])  # not there; of another interpreter, or half written
def test_without_the_native_marshalling_the_library_alone_serves(world, monkeypatch, tmp_path, content):
    seen, general, answer = world
    answer[0] = adacc.OK
    for i, call in enumerate(_every_call()):
        general(True)
        want = _outcome(call), list(seen)
        del seen[:]
        general(False)
        monkeypatch.setattr(adacc, "CALLS_PATH", _broken(tmp_path, content))
        with warnings.catch_warnings(record=True) as told:
            warnings.simplefilter("always")
            assert (_outcome(call), list(seen)) == want
            again = _outcome(call)
        assert again == want[0] and len(told) <= 1  # looked for once
        del seen[:]


def test_the_native_marshalling_carries_the_interpreters_tag():
    assert adacc.CALLS_PATH.endswith("_calls" + sysconfig.get_config_var("EXT_SUFFIX"))


def test_a_build_without_a_c_compiler_goes_on(monkeypatch, tmp_path, capsys):
    from paper_2508_00806_amd import build
    monkeypatch.setattr(build, "CALLS", _broken(tmp_path, b"an older one"))
    monkeypatch.setenv("CC", str(tmp_path / "no-compiler"))
    assert build.build_calls() is None
    assert not os.path.exists(build.CALLS) and "general way" in capsys.readouterr().out


def test_a_workspace_is_handed_over_as_it_is_now(world):
    """The struct that the workspace holds at the time of the call, not one that it held before."""
    seen, general, answer = world
    answer[0] = adacc.OK
    m = adacc.Method(outlier_mode=adacc.OUTLIER_ABS, thresh=1.0, max_outliers=9)
    x, blob, w = torch.zeros(64, dtype=torch.bfloat16), torch.zeros(4096, dtype=torch.uint8), _workspace()
    w.c = adacc.CWorkspace(8192, 1024, 3, 0)
    bare = adacc.Workspace.__new__(adacc.Workspace)
    bare.c = adacc.CWorkspace(12288, 2048, 5, 0)
    for workspace in (w, bare):
        for on in (True, False):
            general(on)
            assert _outcome(lambda: adacc.compress(m, x, blob, workspace, stream=17)) is None
        one, other = seen
        assert one == other and one[1][5] == (workspace.c.device_mem, workspace.c.bytes, workspace.c.epoch, 0)
        del seen[:]
