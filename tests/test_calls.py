"""The choice between the native calls (csrc/bl_calls.cpp) and the ctypes binding, without a GPU: the library and the native
module are stand-ins that record what reaches them."""
import ctypes
import os
import subprocess
import sys
import types

import pytest

from paper_2410_16144_amd import binding as B

STREAM = 0x77


class Recorder:
    """Records (name, arguments) of every call; answers with `answer`."""

    def __init__(self, answer):
        self.seen, self.answer = [], answer

    def __getattr__(self, name):
        def call(*a):
            self.seen.append((name, a))
            return self.answer
        return call


@pytest.fixture
def native_and_library(monkeypatch):
    """A native module that refuses everything, and a library that accepts everything."""
    native, library = Recorder(None), Recorder(B.BL_OK)
    monkeypatch.setattr(B, "_calls", types.SimpleNamespace(launch=native.launch, stream=lambda: STREAM))
    monkeypatch.setattr(B, "_lib", library)
    return native, library


DESC = B.PackedDesc(1, 0, 64, 64, 64, 64, 1024, 0.5, 0.0)
LAUNCHES = [   # which, rows of the ctypes items, what makes them, the entry point
    (B.LAUNCH_GEMV_BATCH, [(1, DESC, 2, 3, 4, 5, 0)], B.make_gemv_items, "bl_gemv_batch"),
    (B.LAUNCH_DECODE_BATCH, [(1, 0, 64, 2, DESC, 3, 0, 0, 0, 0)], B.make_decode_items, "bl_decode_batch"),
    (B.LAUNCH_QUANT_BATCH, [(1, 0, 1, 64, 64, 2, 3, 4)], B.make_quant_items, "bl_quant_act_batch"),
    (B.LAUNCH_TL2_BATCH, [(1, DESC, 2, 3, 0, 5, 0)], B.make_gemv_items, "bl_tl2_gemv_batch"),
]


@pytest.mark.parametrize("which,rows,make,name", LAUNCHES)
def test_items_that_are_no_array_are_launched_through_ctypes(native_and_library, which, rows, make, name):
    """An iterable of tuples, which the ctypes binding turns into an array; it must reach the library, not vanish."""
    native, library = native_and_library
    for items in (rows, iter(rows)):
        library.seen.clear()
        B.launch(which, items, 1, 0)
        (called, args), = library.seen
        assert called == name and args[-1] == STREAM and isinstance(args[0], ctypes.Array) and len(args[0]) == 1
    assert not native.seen


@pytest.mark.parametrize("which,rows,make,name", LAUNCHES)
def test_what_the_native_launch_refuses_goes_through_ctypes(native_and_library, which, rows, make, name):
    native, library = native_and_library
    items = make(rows)
    B.launch(which, items, 1, 0)
    assert [n for n, _ in native.seen] == ["launch"] and [n for n, _ in library.seen] == [name]
    assert library.seen[0][1][0] is items


def test_items_of_another_launch_are_not_read_as_its_own(native_and_library):
    """Wrongly typed items: for ctypes to refuse (here a stand-in); the native call, which only sees memory, is not asked."""
    native, library = native_and_library
    B.launch(B.LAUNCH_GEMV_BATCH, B.make_quant_items(LAUNCHES[2][1]), 1, 0)
    B.launch(B.LAUNCH_ATTN_DECODE, B.make_gemv_items(LAUNCHES[0][1]), 1, 0)
    assert not native.seen and [n for n, _ in library.seen] == ["bl_gemv_batch", "bl_attn_decode"]


@pytest.mark.parametrize("status", [B.BL_ERR_COUNT, B.BL_ERR_ALIGN])
def test_a_status_of_the_native_launch_is_raised(monkeypatch, status):
    native = Recorder(status)
    monkeypatch.setattr(B, "_calls", types.SimpleNamespace(launch=native.launch, stream=lambda: STREAM))
    with pytest.raises(B.BitLinearError) as e:
        B.launch(B.LAUNCH_QUANT_BATCH, B.make_quant_items(LAUNCHES[2][1]), 0)
    assert e.value.status == status and "bl_quant_act_batch failed" in str(e.value)
    assert len(native.seen) == 1


def test_without_the_native_module_everything_goes_through_ctypes(monkeypatch):
    """An installation with the library alone: launches reach it, and the stream comes from torch."""
    torch = pytest.importorskip("torch")
    from paper_2410_16144_amd import build
    library = Recorder(B.BL_OK)
    monkeypatch.setattr(B, "_lib", library)
    monkeypatch.setattr(B, "_calls", None)
    monkeypatch.setattr(build, "calls_path", lambda: os.path.join(build.HERE, "_calls.no-such-torch.so"))
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=STREAM))
    assert B.calls() is False and B.current_stream() == STREAM
    items = B.make_quant_items(LAUNCHES[2][1])
    B.launch(B.LAUNCH_QUANT_BATCH, items, 0)
    (name, args), = library.seen
    assert name == "bl_quant_act_batch" and args[0] is items and args[-1] == STREAM


def test_the_native_module_is_of_the_torch_that_loads_it(monkeypatch):
    """Another torch finds no module instead of a stale one, and the build is not up to date for it."""
    torch = pytest.importorskip("torch")
    from paper_2410_16144_amd import build
    here = build.calls_path()
    assert os.path.dirname(here) == build.HERE and torch.__version__ in here and sys.implementation.cache_tag in here
    monkeypatch.setattr(torch, "__version__", "9.9.9")
    assert build.calls_path() != here and not os.path.exists(build.calls_path())

    class Begins(Exception):
        pass

    def begins(*a, **k):
        raise Begins
    monkeypatch.setattr(build, "_newest_input", lambda: 0)
    monkeypatch.setattr(build, "sources", lambda: [])
    monkeypatch.setattr(subprocess, "check_call", begins)
    with pytest.raises(Begins):
        build.build(force=False)
