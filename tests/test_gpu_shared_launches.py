"""Shape groups that share encoder and product launches equal the same matrices alone.

Up to six groups (more than a launch takes), more matrices than the shared clip passes take,
a group larger than a round between small ones, batches in each, both accumulations.
"""
import pytest
import torch

from paper_2607_04422_amd import workloads
from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu

SETS = {
    "two": [(16, 16), (48, 144), (16, 16)],
    "six": [(16, 16), (48, 144), (144, 48), (272, 400), (64, 64), (128, 1040), (208, 16), (64, 64)],
    "many": [(16, 16)] * 66 + [(48, 80)] * 3 + [(32, 48)] * 62 + [(16, 48)] * 3,
    "large_between": [(48, 144), (1024, 3072), (1024, 3072), (1024, 3072), (80, 80), (144, 272)],
}


@pytest.mark.parametrize("acc32", [False, True])
@pytest.mark.parametrize("name", list(SETS))
def test_groups_equal_alone(name, acc32):
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    flags = F.F_DEFAULT | (F.F_FP32_ACCUM if acc32 else 0)
    ins = [torch.from_numpy(workloads.matrix(r, c, seed=i)).cuda() for i, (r, c) in enumerate(SETS[name])]
    outs = F.fp4root_orthogonalize(ins, steps=3, flags=flags)
    for i, x in list(enumerate(ins))[:: max(1, len(ins) // 20)]:
        assert torch.equal(outs[i], F.fp4root_orthogonalize([x], steps=3, flags=flags)[0]), i
