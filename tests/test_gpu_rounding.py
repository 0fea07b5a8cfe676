"""sqrt_normal and div_normal (mg_device.h) against the compiler's root and
division, and numpy's, over the ranges that their comments state: equal to the
bit, and the root of smaller numbers within one unit in the last place.

Numbers of every exponent of a range with random mantissas, and with mantissas
of all zeros, all ones and their neighbours.  The pairs of a division keep the
divisor, its reciprocal, the dividend and the quotient in range.
"""
import ctypes as C
import os

import numpy as np
import pytest
import torch

from paper_2110_00566_amd import build

pytestmark = pytest.mark.gpu
N = 1 << 22
TYPE = {32: (torch.float32, torch.int32, 23, 127), 64: (torch.float64, torch.int64, 52, 1023)}


def numbers(bits, lo, hi, seed):
    """N positive numbers in [2^lo, 2^hi)."""
    ftype, itype, man, bias = TYPE[bits]
    g = torch.Generator(device="cuda").manual_seed(seed)
    m = torch.randint(0, 1 << man, (N,), dtype=itype, device="cuda", generator=g)
    m[: N // 8] = torch.randint(-2, 3, (N // 8,), dtype=itype, device="cuda", generator=g) % (1 << man)
    e = torch.randint(lo + bias, hi + bias, (N,), dtype=itype, device="cuda", generator=g)
    return ((e << man) | m).view(ftype)


def rounding(bits, a, b):
    assert os.path.exists(build.ROUNDING_LIB), "not built: run python -m paper_2110_00566_amd.build"
    fn = getattr(C.CDLL(build.ROUNDING_LIB), "rounding_f%d" % bits)
    out = torch.empty((4, a.numel()), dtype=a.dtype, device="cuda")
    torch.cuda.synchronize()
    ptr = [C.c_void_p(t.data_ptr()) for t in (a, b)]
    assert fn(ptr[0], ptr[1], C.c_size_t(a.numel()), C.c_void_p(out.data_ptr())) == 0
    return out


@pytest.mark.parametrize("bits,lo,hi,ulp", [(32, -96, 127, 0), (32, -126, -96, 1), (64, -767, 1023, 0),
                                            (64, -1022, -767, 1)])
def test_root(bits, lo, hi, ulp):
    x = numbers(bits, lo, hi, 1)
    itype = TYPE[bits][1]
    root, ref = rounding(bits, x, torch.ones_like(x))[:2]
    assert int((root.view(itype) - ref.view(itype)).abs().max()) <= ulp
    assert np.array_equal(ref.cpu().numpy(), np.sqrt(x.cpu().numpy()))


@pytest.mark.parametrize("bits,blo,bhi,lo,hi", [(32, -126, 126, -100, 126), (64, -1022, 1022, -960, 1022)])
def test_division(bits, blo, bhi, lo, hi):
    # a = q b (1 + O(eps)) for a q of every exponent: any a and any quotient
    a, b = numbers(bits, lo, hi, 2), numbers(bits, blo, bhi, 3)
    q = a / b
    keep = (q >= 2.0 ** lo) & (q < 2.0 ** hi)
    a, b = a[keep], b[keep]
    a[::2] = -a[::2]
    assert a.numel() > N // 4
    quot, ref = rounding(bits, a, b)[2:]
    assert torch.equal(quot, ref)
    assert np.array_equal(ref.cpu().numpy(), a.cpu().numpy() / b.cpu().numpy())


@pytest.mark.parametrize("bits", [32, 64])
def test_special_arguments(bits):
    nan, one = float("nan"), 1.0
    a = torch.tensor([nan, one, nan, 0.0], dtype=TYPE[bits][0], device="cuda")
    b = torch.tensor([one, nan, nan, 3.0], dtype=TYPE[bits][0], device="cuda")
    root, _, quot, _ = rounding(bits, a, b)
    assert torch.isnan(root[0]) and torch.isnan(root[2]) and float(root[1]) == 1.0
    assert torch.isnan(quot[:3]).all() and float(quot[3]) == 0.0
