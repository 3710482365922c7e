"""The AdamW step's quick square roots, quotients and BF16 pairs against the general
operations on the GPU: every binary32 value of the square root's range, every binary32 value
but NaN for the conversion, and 2^32 random quotients per seed."""
import ctypes
import os

import pytest
import torch

from paper_2607_04422_amd import build
from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


def _sweep(name, *args):
    need_gpu()
    if not os.path.exists(build.SWEEPS):
        pytest.fail("libfp4root_sweeps.so is not built (run __graft_entry__.build())")
    lib = ctypes.CDLL(build.SWEEPS)
    out = torch.zeros(2, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    assert getattr(lib, name)(*args, ctypes.c_void_p(out.data_ptr()), None) == 0
    torch.cuda.synchronize()
    bad, which = (int(v) & 0xFFFFFFFF for v in out)
    assert bad == 0, f"{bad} differ, one of them {which:#010x}"


def test_sqrt_every_value():
    u = ctypes.c_uint32
    _sweep("fp4root_sweep_sqrt", u(0x0D800000), u(0x71800000 - 0x0D800000 + 1))   # 2^-100 .. 2^100
    _sweep("fp4root_sweep_sqrt", u(0), u(1))                                      # and zero


def test_bf16_pair_every_value():
    u = ctypes.c_uint32   # each with its negative
    _sweep("fp4root_sweep_bf16", u(0), u(0x7F800001))


@pytest.mark.parametrize("seed", [1, 2])
def test_quotients(seed):
    _sweep("fp4root_sweep_div", ctypes.c_uint64(seed), ctypes.c_uint32(0xFFFFFFFF))
