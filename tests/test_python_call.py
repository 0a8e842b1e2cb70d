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
