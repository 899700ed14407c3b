"""The stream that single-operation calls use: the current one of the current device, by whichever way the installed torch offers."""
import types

import pytest
import torch  # noqa: F401  (before the library: both are to use the HIP runtime that torch brings)

from paper_1901_06773_amd import binding as B


def test_the_public_way_where_the_short_one_is_missing():
    cuda = types.SimpleNamespace(current_stream=lambda: types.SimpleNamespace(cuda_stream=77))
    assert B._stream_ptr(types.SimpleNamespace(_C=types.SimpleNamespace(), cuda=cuda)) == 77
    assert B._stream_ptr(types.SimpleNamespace(_C=types.SimpleNamespace(_cuda_getDevice=lambda: 0), cuda=cuda)) == 77


def test_the_short_way_asks_for_the_current_device():
    c = types.SimpleNamespace(_cuda_getDevice=lambda: 3, _cuda_getCurrentRawStream=lambda d: 100 + d)
    assert B._stream_ptr(types.SimpleNamespace(_C=c)) == 103


def test_errors_of_the_runtime_are_not_swallowed():
    def broken():
        raise RuntimeError("no device")
    c = types.SimpleNamespace(_cuda_getDevice=broken, _cuda_getCurrentRawStream=lambda d: 0)
    with pytest.raises(RuntimeError):
        B._stream_ptr(types.SimpleNamespace(_C=c))
