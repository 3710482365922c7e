"""BF16 path: batches whose library product keeps partial tiles in its scratch.

The scratch is the end of a step's workspace: a margin behind it has to stay untouched
(and keeps an overrun inside the test's own buffer).  Results equal the same matrices one
by one up to the binary32 accumulation of the product, whose order the library chooses by
the batch.
"""
import ctypes

import pytest
import torch

from oracle import ns
from paper_2607_04422_amd import workloads
from tests.gpu_util import need_gpu, np_, rel_fro

pytestmark = pytest.mark.gpu

MARGIN = 128 << 20


def _unit_batch(batch, m, n):
    g = torch.Generator(device="cuda").manual_seed(batch + m)
    x = torch.randn((batch, m, n), generator=g, device="cuda")
    return x / x.flatten(1).double().norm(dim=1).float()[:, None, None]


def _step(F, x):
    b, m, n = x.shape
    lib = F.load()
    need = lib.fp4root_ns_step_workspace(b, m, n, F.F_BF16_PATH)
    ws = torch.full((need + MARGIN,), 0xA5, dtype=torch.uint8, device="cuda")
    y = x.clone()
    p = ctypes.c_void_p
    assert lib.fp4root_ns_step(p(y.data_ptr()), b, m, n, m * n, 3.0, -3.2, 1.2, F.F_BF16_PATH, 0, 0, None,
                               p(ws.data_ptr()), need, None) == 0
    torch.cuda.synchronize()
    assert bool((ws[need:] == 0xA5).all()), (b, m, n)
    return y


@pytest.mark.parametrize("shape", [(3, 16, 48), (3, 256, 512), (16, 144, 11760), (5, 1024, 3072), (8, 3072, 3072),
                                   (3, 3072, 8192)])
def test_step_stays_in_its_scratch(shape):
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    x = _unit_batch(*shape)
    y = _step(F, x)
    for i in range(shape[0]):
        one = _step(F, x[i:i + 1].clone())[0].double()
        # binary32 sums of m products in two orders: m 2^-24 of the sum of magnitudes at most
        assert float((y[i].double() - one).norm() / one.norm()) <= 1e-4, i


def test_batch_of_three_against_the_oracle():
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    mats = [workloads.matrix(*s, seed=i) for i, s in enumerate([(256, 512), (512, 256), (256, 512)])]
    co = [(3.0, -3.2, 1.2)] * 3 + [(1.875, -1.25, 0.375)] * 2
    outs = F.fp4root_orthogonalize([torch.from_numpy(m).cuda() for m in mats], steps=5, coeffs=co,
                                   flags=F.F_CLIP | F.F_BF16_PATH)
    for m, o in zip(mats, outs):   # tolerance: see TOL_BF16 of the single-matrix test (2^-7)
        assert rel_fro(np_(o), ns.orthogonalize(m, co, seed=0, mode="bf16")) <= 2.0 ** -7


def test_grouped_call_equals_matrices_alone():
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    shapes = [(3072, 3072)] * 8 + [(8192, 3072)] * 2 + [(3072, 8192)]
    ins = [torch.from_numpy(workloads.matrix(r, c, seed=7)).cuda() * (1 + i) for i, (r, c) in enumerate(shapes)]
    flags = F.F_DEFAULT | F.F_BF16_PATH
    outs = F.fp4root_orthogonalize(ins, flags=flags)
    for i, x in enumerate(ins):
        alone = F.fp4root_orthogonalize([x], flags=flags)[0].double()
        assert float((outs[i].double() - alone).norm() / alone.norm()) <= 2.0 ** -7, (i, tuple(x.shape))
