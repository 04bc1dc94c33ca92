"""The native marshalling of repeated calls (native/altcall.c) takes, refuses and raises what the calls through ctypes do: every form of every
argument goes through both.  (Without a GPU a call that is taken ends in the library's own status.)"""
import ctypes
import gc
import os
import weakref

import numpy as np
import pytest

import paper_2210_12415_amd as alt
from paper_2210_12415_amd import binding

if binding._native is None:
    pytest.skip("the native module is not built", allow_module_level=True)
if os.path.exists("/dev/kfd"):
    pytest.skip("addresses of no buffer: for machines without a GPU", allow_module_level=True)


class Tensor:
    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        if isinstance(self.at, Exception):
            raise self.at
        return self.at


class Stream:
    def __init__(self, at):
        self.cuda_stream = at


ADDRESSES = [Tensor(64), 128, None, np.int64(256), Tensor(RuntimeError("no storage")), Tensor(np.int64(64)), "text", 1.5, -1, 1 << 64, True]
STREAMS = [0, Stream(64), Stream(np.int64(64)), np.int32(0), "text", -1, ctypes.c_void_p(0)]
SIZES = [0, 1 << 40, -1, 1 << 64, np.int64(8), ctypes.c_size_t(8), None, 1.5, True]
DTYPES = [alt.BF16, np.int32(1), 256, -1, 1 << 64, None, "1", True, ctypes.c_int(1)]
LAYOUT = alt.layout_parse("NCHW->NHWC")
SHAPES = [(1, 8, 4, 4), [1, 8, 4, 4], np.array([1, 8, 4, 4]), (1, 8, 4), (1, 8, 4, np.int64(4)), (1, 8, 4, -4), (1, 8, 4, 1 << 63), (1, 8, 4, 4.5), 5, ()]

CALLS = {
    "layout_transform": (dict(dtype=alt.BF16, shape=(1, 8, 4, 4), src_layout=LAYOUT, src=Tensor(64), dst_layout=LAYOUT, dst=Tensor(128), stream=0),
                         dict(dtype=DTYPES, shape=SHAPES, src=ADDRESSES, dst=ADDRESSES, stream=STREAMS, src_layout=["NCHW->NHWC", None, alt.gemm_desc(1, 1, 1)])),
    "eltwise_add": (dict(dtype=alt.BF16, numel=8, a=Tensor(64), b=Tensor(128), y=Tensor(192), stream=0),
                    dict(dtype=DTYPES, numel=[8, 0, -8, np.int64(8), ctypes.c_int64(8), 1 << 64, 1.5, None], a=ADDRESSES, y=ADDRESSES, relu=[True, 1, 0, "", None, np.True_], stream=STREAMS)),
    "gemm": (dict(d=alt.gemm_desc(8, 8, 8), A=Tensor(64), B=Tensor(128), C=Tensor(192), stream=0),
             dict(d=[None, alt.conv_desc(1, 8, 8, 8, 8, 1, 1), 64], A=ADDRESSES, C=ADDRESSES, workspace=ADDRESSES, ws_bytes=SIZES, stream=STREAMS)),
}
for name in ("conv2d", "conv2d_prepared", "conv2d_transpose", "conv3d", "conv3d_transpose"):
    d = alt.conv3d_desc(1, 8, 8, 8, 8, 8, 1, 1, 1) if "3d" in name else alt.conv_desc(1, 8, 8, 8, 8, 1, 1)
    CALLS[name] = (dict(d=d, x=Tensor(64), w=Tensor(128), y=Tensor(192), stream=0),
                   dict(d=[None, alt.gemm_desc(8, 8, 8)], x=ADDRESSES, bias=ADDRESSES, y=ADDRESSES, workspace=ADDRESSES, ws_bytes=SIZES, stream=STREAMS))


def outcome(h, name, kw):
    try:
        r = getattr(h, name)(**kw)
        return r() if name == "conv2d_prepared" else r
    except Exception as e:
        return type(e), str(e)


@pytest.mark.parametrize("name", list(CALLS))
def test_native_and_ctypes_calls_agree(name, monkeypatch):
    h = alt.Handle()
    base, forms = CALLS[name]
    quick = {n: getattr(binding, n) for n in dir(binding) if n.startswith("_quick_")}
    taken = []
    for key, values in list(forms.items()) + [(None, [None])]:
        for v in values:
            kw = dict(base, **({key: v} if key else {}))
            for n, f in quick.items():
                monkeypatch.setattr(binding, n, lambda *a, f=f: taken.append(f(*a)) or taken[-1])
            native = outcome(h, name, kw)
            for n in quick:
                monkeypatch.setattr(binding, n, binding._not_taken)
            assert native == outcome(h, name, kw), (key, v)
    assert any(t is not None for t in taken) and any(t is None for t in taken)


def test_prepared_call_keeps_its_arguments():
    h = alt.Handle()
    x = Tensor(64)
    alive = weakref.ref(x)
    run = h.conv2d_prepared(alt.conv_desc(1, 8, 8, 8, 8, 1, 1), x, Tensor(128), Tensor(192), stream=0)
    del x
    gc.collect()
    assert alive() is not None
    with pytest.raises(alt.AltError):
        run()
    with pytest.raises(TypeError):
        run(1)
    del run
    gc.collect()
    assert alive() is None


@pytest.mark.parametrize("native", [True, False], ids=["native", "ctypes"])
@pytest.mark.parametrize("several", [False, True], ids=["one", "several"])
def test_prepared_call_keeps_its_handle(native, several, monkeypatch):
    """A prepared call outlives the caller's reference to the Handle and to its tensors; after close() it finds no handle."""
    if not native:
        monkeypatch.setattr(binding, "_quick_prepare", binding._not_taken)

    def prepare(h, x):
        kw = dict(d=alt.conv_desc(1, 8, 8, 8, 8, 1, 1), x=x, w=Tensor(128), y=Tensor(192), stream=0)
        run = h.conv2d_multi_prepared([kw, kw]) if several else h.conv2d_prepared(**kw)
        kw["x"] = None
        return run

    h, x = alt.Handle(), Tensor(64)
    alive = weakref.ref(h), weakref.ref(x)
    run = prepare(h, x)
    del h, x
    gc.collect()
    assert all(a() is not None for a in alive)
    with pytest.raises(alt.AltError, match="no GPU"):
        run()
    del run
    gc.collect()
    assert all(a() is None for a in alive)

    h = alt.Handle()
    run = prepare(h, Tensor(64))
    h.close()
    with pytest.raises(alt.AltError, match="invalid argument"):
        run()


@pytest.mark.parametrize("name", list(CALLS))
def test_interrupts_are_raised_at_once(name):
    """An interrupt inside an argument's own code ends the call; ctypes does not ask the argument again."""
    asked = []

    class Interrupted:
        def data_ptr(self):
            asked.append(1)
            if len(asked) == 1:
                raise KeyboardInterrupt
            return 64

    base = CALLS[name][0]
    kw = dict(base, **{next(k for k in ("x", "A", "a", "src") if k in base): Interrupted()})
    with pytest.raises(KeyboardInterrupt):
        getattr(alt.Handle(), name)(**kw)
    assert len(asked) == 1
