"""Products whose chained groups span several 64-element stages, against the oracle.

Contractions of at least 1024 elements take chain bounds over aligned runs of one, two and
four stages, kept per 32 rows.  The shapes put every edge in: the first such contraction,
stage counts that are not multiples of two or four, a partial last stage, row counts that
are not multiples of 32 or 64, a contraction below the limit on one side only, more than 64
stages (a second window of decisions) and more than 512 (past the last window, where every
block folds).  Every product is exact, so a step must equal the oracle's bit for bit in both
tile forms.
"""
import numpy as np
import pytest
import torch

from oracle import ns, rht
from paper_2607_04422_amd import workloads
from tests.gpu_util import need_gpu, np_
from tests.test_chain_levels import mixed_matrix

pytestmark = pytest.mark.gpu

SHAPES = [(16, 1024), (48, 1040), (272, 1104), (112, 2000), (1040, 1088), (80, 4240)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("form", [1, 2])
@pytest.mark.parametrize("scaled", [False, True])
def test_step_over_runs_of_stages(shape, form, scaled):
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    m, n = shape
    x = workloads.matrix(m, n, seed=90 + m % 7)
    x = (x / np.linalg.norm(x.astype(np.float64))).astype(np.float32)
    if scaled:   # block exponents that vary along the contraction: most stages fail their own bound
        x *= np.exp2(np.random.default_rng(5).integers(-6, 7, size=(1, n // 16)).repeat(16, axis=1)).astype(np.float32)
    ref = ns.ns_step_nvfp4(x, 3.0, -3.2, 1.2, rht.step_signs(7, 2), True)
    t = torch.from_numpy(x).cuda()
    prev = F.fp4root_set_product_tiling(form)
    try:
        F.fp4root_ns_step(t, 3.0, -3.2, 1.2, seed=7, step=2)
        torch.cuda.synchronize()
    finally:
        F.fp4root_set_product_tiling(prev)
    got = np_(t)
    assert np.array_equal(got, ref), f"{np.count_nonzero(got != ref)} of {ref.size} differ"


@pytest.mark.parametrize("shape", [(272, 1104), (112, 2000), (48, 4240), (16, 32848)])
@pytest.mark.parametrize("form", [1, 2])
def test_step_with_every_kind_of_run(shape, form):
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    x = mixed_matrix(*shape)   # its stages' bounds: see test_mixed_matrix_has_every_outcome
    ref = ns.ns_step_nvfp4(x, 3.0, -3.2, 1.2, rht.step_signs(7, 2), True)
    t = torch.from_numpy(x).cuda()
    prev = F.fp4root_set_product_tiling(form)
    try:
        F.fp4root_ns_step(t, 3.0, -3.2, 1.2, seed=7, step=2)
        torch.cuda.synchronize()
    finally:
        F.fp4root_set_product_tiling(prev)
    got = np_(t)
    assert np.array_equal(got, ref), f"{np.count_nonzero(got != ref)} of {ref.size} differ"
