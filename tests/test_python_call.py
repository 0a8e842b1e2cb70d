"""The extension module behind the binding's calls (csrc/python_call.cpp), without a GPU: every argument of every entry point arrives at its
place, as ctypes itself would pass it."""
import ctypes

import pytest

from paper_1705_05249_amd import gemm as G


def test_every_argument_arrives():
    import torch
    L, call = G.lib(), G._native()
    names = [name for name in G.EXPORTS if hasattr(call, name)]
    assert len(names) == 19
    try:
        for name in names:
            types, seen, args, expected = getattr(L, name).argtypes, [], [], []
            for i, t in enumerate(types):
                if t is ctypes.c_size_t and types[i - 1] is ctypes.c_void_p:
                    expected.append(args[-1].numel() * args[-1].element_size())
                elif t is ctypes.c_float:
                    args.append(0.5 + i)
                    expected.append(0.5 + i)
                elif t is ctypes.c_void_p and i + 1 < len(types):
                    args.append(torch.zeros(3 + i, dtype=torch.float16))
                    expected.append(args[-1].data_ptr())
                else:
                    args.append((1 << 40) + i if t is ctypes.c_int64 else 1000 + i)         # (the last pointer: a stream's address)
                    expected.append(args[-1])
            made = ctypes.CFUNCTYPE(ctypes.c_int32, *types)(lambda *a: seen.extend(a) or -7)
            call.bind({name: ctypes.cast(made, ctypes.c_void_p).value}, G._stream_calls)
            assert getattr(call, name)(*args) == -7
            assert seen == expected, name
            with pytest.raises(TypeError):
                getattr(call, name)(*args[:-1])
            with pytest.raises(TypeError):
                getattr(call, name)("layout", *args[1:])
    finally:
        G._call = None
        G._native()
    assert G.mg_sgemm(0, G.MG_NO_TRANS, G.MG_NO_TRANS, 4, 4, 4, 1, None, 4, None, 4, 0, None, 4, None, 0, check=False) == -1


def test_no_workspace_and_stream_objects():
    class Stream:
        cuda_stream = 77

    L, call, seen = G.lib(), G._native(), []
    made = ctypes.CFUNCTYPE(ctypes.c_int32, *L.mg_hgemv.argtypes)(lambda *a: seen.append(a) or 0)
    try:
        call.bind({"mg_hgemv": ctypes.cast(made, ctypes.c_void_p).value}, G._stream_calls)
        G.mg_hgemv(G.MG_COL_MAJOR, G.MG_NO_TRANS, 2, 3, 1.0, 4096, 2, 8192, 1, 0.0, 12288, 1, None, Stream())
    finally:
        G._call = None
        G._native()
    (args,) = seen
    assert args[5] == 4096 and args[7] == 8192 and args[10] == 12288 and args[12:] == (None, 0, 77)


def test_ctypes_scalars_are_taken_as_ctypes_takes_them():
    """integers and floats of ctypes for any scalar argument; what arrives is their value"""
    L, call, seen = G.lib(), G._native(), []
    good = (G.MG_COL_MAJOR, G.MG_NO_TRANS, G.MG_NO_TRANS, 0, 3, 5, 1.0, None, 1, None, 5, 0.0, None, 1)
    try:
        for i, (value, t) in enumerate(zip(good, L.mg_hgemm.argtypes)):
            if t is not ctypes.c_void_p:
                assert G.mg_hgemm(*good[:i], t(value), *good[i + 1:], None, 0) == 0
        # (an output without rows: nothing runs)  an illegal value arrives as such
        assert G.mg_hgemm(ctypes.c_int(0), *good[1:], None, 0, check=False) == -1
        assert G.mg_hgemm(good[0], good[1], good[2], ctypes.c_int64(-1), *good[4:], None, 0, check=False) == -4
    finally:
        G._call = None
        G._native()


def test_wrong_types_raise_what_ctypes_raises():
    args = (G.MG_COL_MAJOR, G.MG_NO_TRANS, 2, 3, 1.0, 4096, 2, 8192, 1, 0.0, 12288, 1)
    for i, wrong in ((0, "layout"), (2, 2.0), (4, "one"), (2, None), (4, 10 ** 400)):
        with pytest.raises(ctypes.ArgumentError):
            G.mg_sgemv(*args[:i], wrong, *args[i + 1:], None, 0)
        with pytest.raises(TypeError):
            G.mg_sgemv(*args[:i], wrong, *args[i + 1:], None, 0)
    with pytest.raises(AttributeError):
        G.mg_sgemv(*args[:5], 2.5, *args[6:], None, 0)              # no address


def test_missing_extension_says_what_to_build(monkeypatch, tmp_path):
    monkeypatch.setattr(G, "_call", None)
    monkeypatch.setattr(G, "CALL_PATH", str(tmp_path / "_mg_call.so"))
    with pytest.raises(RuntimeError, match="build it first"):
        G.mg_sgemm(0, G.MG_NO_TRANS, G.MG_NO_TRANS, 4, 4, 4, 1, None, 4, None, 4, 0, None, 4, None, 0, check=False)
