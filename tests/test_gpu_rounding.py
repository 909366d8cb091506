"""The tracker's square root and reciprocal are the correctly rounded ones for every
mantissa.  That follows from their Newton steps only together with what the chip's
approximations start them from, so all 2^23 mantissas are compared with IEEE
arithmetic on the host: at exponents of both parities (the root repeats every two,
the reciprocal every one), at the ends of the range that the tracker gives them
(pivots in [2^-90, 2^120], of which the reciprocal takes the roots), and at the
whole range that the source names.  A Newton step from the wrong neighbour would
show at the mantissa of all ones."""
import ctypes
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "librounding.so")
EXPONENTS = [-98, -97, -90, -89, -45, -44, -1, 0, 1, 2, 23, 24, 59, 60, 118, 119]


@pytest.fixture(scope="module")
def rounding():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib = ctypes.CDLL(LIB)   # built by __graft_entry__.build()
    lib.rounding.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_int, ctypes.c_void_p]
    lib.rounding.restype = ctypes.c_int

    def call(x):
        n = len(x)
        dev, root, rcp = torch.from_numpy(x).cuda(), torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
        assert lib.rounding(dev.data_ptr(), root.data_ptr(), rcp.data_ptr(), n,
                            torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        return root.cpu().numpy(), rcp.cpu().numpy()

    return call


@pytest.mark.parametrize("exponent", EXPONENTS)
def test_every_mantissa(rounding, exponent):
    print(f"case rounding 2^{exponent}", flush=True)
    bits = np.arange(1 << 23, dtype=np.uint32) | np.uint32((exponent + 127) << 23)
    x = bits.view(np.float32)
    root, rcp = rounding(x)
    assert np.array_equal(root, np.sqrt(x))
    assert np.array_equal(rcp, np.float32(1.0) / x)


def test_the_upper_end(rounding):
    x = np.array([2.0 ** 120, 2.0 ** 60, 2.0 ** -90], np.float32)
    root, rcp = rounding(x)
    assert np.array_equal(root, np.sqrt(x)) and np.array_equal(rcp, np.float32(1.0) / x)
