"""Argument marshalling of the Python binding, on the CPU: the library is a
stub that records the call, or the built one up to its argument checks."""
import os
import types

import numpy as np
import pytest
import torch

from paper_2607_01065_amd import gsrq as B


class _Lib:
    """Stands in for the library: records encode_prepared's arguments."""

    def gsrq_encode_prepared(self, sh, x, dtype, ldx, prepared, codes, residual, stream):
        s = sh._obj
        self.call = (s.N, s.D, s.d, s.K, s.M, ldx, stream)
        return B.GSRQ_OK


def _stream(handle):
    return types.SimpleNamespace(cuda_stream=handle)


@pytest.mark.parametrize("number", [int, np.int64, np.int32])
@pytest.mark.parametrize("d,K,M,words", [(8, 256, 1, 2), (8, 256, 3, 6), (4, 2, 1, 1), (8, 32, 2, 3)])
def test_append_takes_any_integers(monkeypatch, number, d, K, M, words):
    """A Prepared rebuilt from saved arrays holds numpy integers."""
    lib = _Lib()
    monkeypatch.setattr(B, "_lib", lib)
    prep = B.Prepared(torch.zeros(256, dtype=torch.uint8), 64, number(d), number(K), number(M))
    codes, _ = B.encode_prepared(torch.zeros((5, 64), dtype=torch.float16), prep, stream=_stream(16))
    assert tuple(codes.shape) == (5, words) and lib.call == (5, 64, d, K, M, 64, 16)


@pytest.mark.skipif(not os.path.exists(B.LIB_PATH), reason="libgsrq.so not built")
@pytest.mark.parametrize("d,K,M", [(0, 256, 1), (-8, 256, 1), (8, 0, 1), (8, 200, 1), (8, 256, 0), (7, 256, 1)])
def test_append_refuses_shapes_through_the_library(d, K, M):
    prep = B.Prepared(torch.zeros(256, dtype=torch.uint8), 64, d, K, M)
    with pytest.raises(B.GsrqError) as e:
        B.encode_prepared(torch.zeros((5, 64), dtype=torch.float16), prep, stream=_stream(0))
    assert e.value.status == B.GSRQ_E_ARG


def test_append_stream_without_private_calls(monkeypatch):
    lib = _Lib()
    monkeypatch.setattr(B, "_lib", lib)
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: _stream(1234))
    prep = B.Prepared(torch.zeros(256, dtype=torch.uint8), 64, 8, 256, 1)
    B.encode_prepared(torch.zeros((5, 64), dtype=torch.float16), prep)
    assert lib.call[-1] == 1234


def test_other_calls_ask_for_the_current_stream(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: _stream(77))
    assert B._stream_handle(None) == 77
    assert B._stream_handle(_stream(5)) == 5 and B._stream_handle(_stream(0)) is None
