"""CPU tests of the host conversions of 16-bit storage (encode_values / decode_values of the
library), in the default floating-point mode and with the thread flushing denormals to zero, as
torch.set_flush_denormal and libraries built with fast math leave it: the values of binary16 are
normal doubles, so the mode must not show."""
import ctypes

import numpy as np
import pytest

from paper_1912_09327_amd import _capi as C

F16S, BF16S = C.PRECISIONS["f16s"], C.PRECISIONS["bf16s"]
DECODE = "_ZN4lbt113decode_valuesEiPKvmdPd"  # lbt1::decode_values(int, void const*, size_t, double, double*)
ENCODE = "_ZN4lbt113encode_valuesEiPKdmdPv"  # lbt1::encode_values(int, double const*, size_t, double, void*)


def _decode(prec, codes, scale=1.0):
    f = getattr(C.lib, DECODE)
    f.restype, f.argtypes = None, [ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_double, ctypes.c_void_p]
    codes = np.ascontiguousarray(codes, np.uint16)
    out = np.empty(codes.size)
    f(prec, codes.ctypes.data, codes.size, scale, out.ctypes.data)
    return out


def _encode(prec, values, inv_scale=1.0):
    f = getattr(C.lib, ENCODE)
    f.restype, f.argtypes = None, [ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_double, ctypes.c_void_p]
    values = np.ascontiguousarray(values, np.float64)
    out = np.empty(values.size, np.uint16)
    f(prec, values.ctypes.data, values.size, inv_scale, out.ctypes.data)
    return out


@pytest.fixture(params=[False, True], ids=["default", "flush denormals"])
def flushing(request):
    import torch
    if request.param and not torch.set_flush_denormal(True):
        pytest.skip("this CPU cannot flush denormals")
    yield request.param
    torch.set_flush_denormal(False)


def test_every_half_code_decodes(flushing):
    codes = np.arange(65536, dtype=np.uint16)
    got = _decode(F16S, codes)
    import torch
    torch.set_flush_denormal(False)
    ref = codes.view(np.float16).astype(np.float64)
    nan = np.isnan(ref)
    assert np.array_equal(np.isnan(got), nan)
    assert np.array_equal(got[~nan].view(np.uint64), ref[~nan].view(np.uint64))  # the sign of zero too


def test_half_codes_round_trip(flushing):
    """Every code but the NaNs, its neighbours' midpoints and both sides of them, and what rounds
    to infinity or to zero."""
    codes = np.arange(0x7c01, dtype=np.uint16)
    v = codes.view(np.float16).astype(np.float64)
    assert np.array_equal(_encode(F16S, v), codes) and np.array_equal(_encode(F16S, -v), codes | 0x8000)
    v[-1] = 65536.0  # where the next value would lie
    mid = 0.5 * (v[:-1] + v[1:])
    even = codes[:-1] + (codes[:-1] & 1)
    assert np.array_equal(_encode(F16S, mid), even)
    assert np.array_equal(_encode(F16S, np.nextafter(mid, 0)), codes[:-1])
    assert np.array_equal(_encode(F16S, np.nextafter(mid, np.inf)), codes[1:])
    for big in (65536.0, 1e10, 1e300, np.inf):
        assert list(_encode(F16S, [big, -big])) == [0x7c00, 0xfc00]
    assert list(_encode(F16S, [1e-30, -1e-30, 0.0, -0.0])) == [0, 0x8000, 0, 0x8000]
    assert _encode(F16S, [np.nan])[0] & 0x7fff == 0x7e00


def test_normal_bfloat16_codes(flushing):
    """The normal values of bfloat16 (its subnormals are subnormal floats, which the mode is about)."""
    codes = np.concatenate([np.arange(0x80, 0x7f81), np.arange(0x8080, 0xff81), [0, 0x8000]]).astype(np.uint16)
    ref = (codes.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    assert np.array_equal(_decode(BF16S, codes).view(np.uint64), ref.view(np.uint64))
    assert np.array_equal(_encode(BF16S, ref), codes)
