"""The short square root of the Metropolis-Hastings and image moves against
the library's and the exact one, over every float that its comment claims
(Box-Muller's arguments lie between 1.1e-7 and 33)."""
import ctypes as C
import os

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi", [(0x0F800000, 0x42800000), (0, 0)])   # [2^-96, 64]; +0
def test_every_float_gives_the_correctly_rounded_root(lo, hi):
    import torch
    from tests.pins import build
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    if not os.path.exists(build.LIB):
        build.build()
    lib = C.CDLL(build.LIB)
    lib.check_sqrt_normal.argtypes = [C.c_uint, C.c_uint, C.c_void_p, C.c_void_p]
    differ = torch.zeros(2, dtype=torch.int64, device="cuda")
    assert lib.check_sqrt_normal(lo, hi - lo + 1, C.c_void_p(differ.data_ptr()),
                                 C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert differ.tolist() == [0, 0]
