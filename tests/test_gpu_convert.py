"""The operand conversions (one value and packed pairs, by the chip's own instructions) against integer
definitions: fp32 -> bf16 round to nearest even with NaN kept NaN, fp32 -> fp16 round to nearest even,
saturating at +-65504 (a NaN becomes -65504).  Every upper half of an fp32 word is met with lower halves around
the rounding points of both formats, so that all exponents, signs, subnormals, infinities, halfway cases
and the fp16 saturation are among the inputs, each as lower and as upper value of a pair."""
import ctypes as C
import os

import numpy as np
import pytest

import paper_2502_02175_amd as V

SAFE = os.path.join(os.path.dirname(V.lib_path()), "libvlac_safe.so")


def bf16_bits(u):
    u = u.astype(np.uint64)
    nan = (u & 0x7fffffff) > 0x7f800000
    return np.where(nan, (u >> 16) | 0x40, (u + 0x7fff + ((u >> 16) & 1)) >> 16).astype(np.uint16)


def f16_bits(u):
    """Round to nearest even in integers: value = m 2^e with m the 24-bit significand."""
    u = u.astype(np.int64)
    sign, mag = (u >> 31) << 15, u & 0x7fffffff
    exp = np.maximum(mag >> 23, 1)
    m = (mag & 0x7fffff) | np.where(mag >> 23 > 0, 1 << 23, 0)
    # a fp16 unit in the last place is 2^(max(e, -14) - 10); the significand's is 2^(e - 23), e = exp - 127
    shift = np.minimum(13 + np.maximum(-14 - (exp - 127), 0), 40)
    half = np.int64(1) << (shift - 1)
    low = m & ((np.int64(1) << shift) - 1)
    q = m >> shift
    q = q + ((low > half) | ((low == half) & (q & 1 == 1)))
    base = np.maximum(exp - 127 + 15, 1)          # exponent field of a normal result; subnormal: 1, less the hidden bit
    out = ((base - 1) << 10) + q                  # (q holds the hidden bit where there is one; a carry moves on by itself)
    out = np.where(mag > 0x477fe000, 0x7bff, out)  # 65504
    out = (sign | out).astype(np.int64)
    return np.where(mag > 0x7f800000, 0xfbff, out).astype(np.uint16)


@pytest.mark.gpu
def test_conversions_bit_for_bit():
    import torch
    lows = [0x0000, 0x0001, 0x0fff, 0x1000, 0x1001, 0x1fff, 0x2000, 0x2fff, 0x3000, 0x3001, 0x5000, 0x7000, 0x7fff, 0x8000, 0x8001,
            0x9000, 0xb000, 0xd000, 0xefff, 0xf000, 0xf001, 0xffff]
    u = ((np.arange(65536, dtype=np.uint32)[:, None] << 16) | np.array(lows, dtype=np.uint32)).reshape(-1)
    signalling = ((u & 0x7fffffff) > 0x7f800000) & (u & 0x400000 == 0)
    u = np.random.default_rng(0).permutation(u[~signalling])  # (no arithmetic returns a signalling NaN)
    n = len(u)
    x = torch.tensor(u.view(np.int32), device="cuda:0")
    out = [torch.zeros(n, dtype=t, device="cuda:0") for t in (torch.int16, torch.int16, torch.int32, torch.int32)]
    f = C.CDLL(SAFE).vlac_convert_check
    f.restype = C.c_int
    assert f(C.c_void_p(x.data_ptr()), C.c_int(n), *(C.c_void_p(o.data_ptr()) for o in out), C.c_void_p(0)) == 0
    torch.cuda.synchronize()
    bf, h = (o.cpu().numpy().view(np.uint16) for o in out[:2])
    bf2, h2 = (o.cpu().numpy().view(np.uint32) for o in out[2:])
    for got, pair, want in ((bf, bf2, bf16_bits(u)), (h, h2, f16_bits(u))):
        bad = np.flatnonzero(got != want)
        assert not len(bad), (hex(u[bad[0]]), hex(got[bad[0]]), hex(want[bad[0]]))
        assert np.array_equal(pair & 0xffff, want)
        assert np.array_equal(pair >> 16, want[::-1])


@pytest.mark.gpu
def test_the_swiglu_quotient_is_the_division_for_every_value():
    """x / (1 + e^-x) by the chip's reciprocal and one step from it, with a scaled one beyond +-87, over all 2^32 fp32 patterns
    (signed zeros, subnormals, denominators up to infinity, infinities, NaN), against the compiler's IEEE division in the same kernel; and that
    division against numpy's, over every 4099th value and all of the denominators above 2^126."""
    import torch
    f = C.CDLL(SAFE).vlac_silu_check
    f.restype = C.c_int
    differ = torch.tensor([0, -1], dtype=torch.int32, device="cuda:0")
    n = 1 << 28
    y, got = (torch.empty(n, dtype=torch.float32, device="cuda:0") for _ in range(2))
    kept = []
    for part in range(16):
        first = part * n
        assert f(C.c_uint32(first), C.c_int(n), C.c_void_p(y.data_ptr()), C.c_void_p(got.data_ptr()),
                 C.c_void_p(differ.data_ptr()), C.c_void_p(0)) == 0
        torch.cuda.synchronize()
        i = torch.arange(0, n, 4099, device="cuda:0")
        if first <= 0xc2ae0000 < first + n:  # -87 .. -89: e^-x of 2^125.5 .. infinity
            i = torch.cat([i, torch.arange(0xc2ae0000 - first, 0xc2b20000 - first, device="cuda:0")])
        kept.append(((i + first).cpu().numpy().astype(np.uint32), y[i].cpu().numpy(), got[i].cpu().numpy()))
    count, least = (int(v) & 0xffffffff for v in differ.cpu())
    x, y, got = (np.concatenate(k) for k in zip(*kept))
    x = x.view(np.float32)
    with np.errstate(all="ignore"):
        want = x / y
    bad = (got.view(np.uint32) != want.view(np.uint32)) & ~(np.isnan(got) & np.isnan(want))
    assert count == 0, (count, hex(least), float(np.array([least], np.uint32).view(np.float32)[0]))
    assert not bad.any(), (x[bad][:4], y[bad][:4], got[bad][:4], want[bad][:4])


def test_the_integer_definitions_are_numpy_s():
    rng = np.random.default_rng(1)
    u = rng.integers(0, 2 ** 32, 400000, dtype=np.uint64).astype(np.uint32)
    x = u.view(np.float32)
    fin = np.isfinite(x) & (np.abs(x) <= 65504)
    assert np.array_equal(f16_bits(u)[fin], x[fin].astype(np.float16).view(np.uint16))
