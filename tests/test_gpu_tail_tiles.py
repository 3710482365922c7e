"""A launch whose last round is cut into 64 x 64 tiles gives the same bits as launches that
take one tile size throughout.

90 matrices of 272 x 400 make 540 Gram tiles (512 + 28) and 1080 update tiles (2 x 512 + 56)
of 128 x 128 with ragged edges; three matrices of 1024 x 1088 beside them put several
products into one Gram launch, with the shorter contraction in the tail.
"""
import numpy as np
import pytest
import torch

from oracle import ns
from paper_2607_04422_amd import workloads
from tests.gpu_util import need_gpu, np_

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extra", [0, 3])
def test_cut_tail_equals_uniform_tiles(extra):
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    base = [workloads.matrix(272, 400, seed=40 + i) for i in range(6)]
    ins = [torch.from_numpy(base[i % 6] * np.float32(1 + i // 6)).cuda() for i in range(90)]
    ins += [torch.from_numpy(workloads.matrix(1024, 1088, seed=60 + i)).cuda() for i in range(extra)]
    runs = []
    for mode in (0, 1, 2):
        prev = F.fp4root_set_product_tiling(mode)
        try:
            runs.append([np_(o) for o in F.fp4root_orthogonalize(ins, steps=2)])
        finally:
            F.fp4root_set_product_tiling(prev)
    for i, (a, b, c) in enumerate(zip(*runs)):
        assert np.array_equal(a, b) and np.array_equal(a, c), f"matrix {i}"
    ref = ns.orthogonalize(np_(ins[0]), F.fp4root_default_coeffs(272, 400, 2), seed=0)
    assert np.array_equal(runs[0][0], ref)
