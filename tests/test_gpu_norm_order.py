"""A matrix's norm does not depend on the matrices beside it.

The first element is L and the others are small enough that a binary64 sum with L^2 drops
each one's square, so how many of them are added to L^2 one by one, and how many are summed
apart first, shows in the last place of the sum; eps puts the inverse norm next to a
binary32 rounding boundary, so that one last place of the sum decides the result.  (The pairs
separate sums over 512 16-byte quads of the matrix from sums over 2048.)
"""
import numpy as np
import pytest
import torch

from oracle import ns
from paper_2607_04422_amd import workloads
from tests.gpu_util import need_gpu, np_

pytestmark = pytest.mark.gpu

SMALL = float.fromhex("0x1.650decp-27")
PLAIN = [("0x1.377214p+0", "0x1.7c744ap-28"), ("0x1.3f03f4p+0", "0x1.551b3p-27"), ("0x1.467f38p+0", "0x1.0c5db2p-28"),
         ("0x1.3fd07ap+0", "0x1.7c11p-28"), ("0x1.1453e6p+0", "0x1.d2e174p-28")]
CLIPPED = [("0x1.2e5a4cp+0", "0x1.05cd3p-30"), ("0x1.2f01b6p+0", "0x1.5622fap-28"), ("0x1.49d5f8p+0", "0x1.c4410ep-28"),
           ("0x1.5018520p+0", "0x1.e7c276p-28"), ("0x1.5965fcp+0", "0x1.63b20cp-28")]


@pytest.mark.parametrize("count", [2, 40, 128, 200])
@pytest.mark.parametrize("clip", [False, True])
def test_rounding_boundary(clip, count):
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    for large, eps in (CLIPPED if clip else PLAIN):
        x = torch.full((512, 512), SMALL, device="cuda")
        x[0, 0] = float.fromhex(large)
        if clip:
            x[0, 1] = 2.0   # the quantile: the norm's sum over the other elements, then 4
        kw = dict(steps=0, eps=float.fromhex(eps), clip_quantile=1.0, flags=F.F_CLIP if clip else 0)
        alone = F.fp4root_orthogonalize([x], **kw)[0]
        for i, o in enumerate(F.fp4root_orthogonalize([x] * count, **kw)):
            assert torch.equal(o, alone), (i, large)


@pytest.mark.parametrize("flags", [0, 1])
def test_batches_and_strides(flags):
    """Random matrices with 1 to 4 parts and a ragged last one, rows contiguous or not."""
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    for r, c in [(16, 16), (48, 176), (272, 144), (336, 400), (128, 1040)]:
        for i in range(3):
            m = torch.from_numpy(workloads.matrix(r, c, seed=i)).cuda()
            buf = torch.zeros((r, c + 16), device="cuda")
            buf[:, :c] = m
            alone = F.fp4root_orthogonalize([m], steps=0, flags=flags)[0]
            many = F.fp4root_orthogonalize([m, buf[:, :c]] * 64 + [m], steps=0, flags=flags)
            for o in many:
                assert torch.equal(o, alone), (r, c, i)
            ref, tall, _ = ns.prepare(np_(m), clip_on=bool(flags))
            assert np.array_equal(np_(alone), ref.T if tall else ref)
