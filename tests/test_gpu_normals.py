"""The FP64 normals' quotient, root, logarithm, sine and cosine have the bits
of the IEEE expressions that they stand for, and the resamplers' FP32 logarithm
keeps well inside the margin in which they ask the FP64 one, at every 32-bit
word (tests/helpers/normals_check.hip)."""
import ctypes
import os
import struct

import pytest

from helpers import NORMALS_CHECK, build_normals_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,sigma", [(0.05, 0.1), (0.01, 0.3), (0.037, 1.0)])
def test_every_word(h, sigma):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lib = ctypes.CDLL(NORMALS_CHECK if os.path.exists(NORMALS_CHECK) else build_normals_check())
    lib.normals_check.argtypes = [ctypes.c_double, ctypes.c_double, ctypes.c_void_p]
    out = (ctypes.c_uint64 * 7)()
    assert lib.normals_check(h, sigma * h ** 0.5, out) == 0
    assert list(out[:6]) == [0] * 6
    far = struct.unpack("d", struct.pack("Q", out[6]))[0]
    assert far < 4e-6, far  # a fifth of the margin
