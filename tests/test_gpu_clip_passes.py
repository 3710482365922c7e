"""The collecting clip passes against the oracle's quantile and norm, bit for bit.

The second pass appends candidate elements to per-wave segments; the last reads only those.
Cases: one tile and many, a last tile of a few quads (its segments may be too short and the
wave reads the matrix again), rows that are not contiguous, tall matrices, quantiles at both
ends (ranks lo and lo + 1 in different bins), every element a candidate (constant
magnitudes), zeros, and more matrices than one chunk holds.
"""
import numpy as np
import pytest
import torch

from oracle import ns
from oracle.quantile import clip_threshold
from paper_2607_04422_amd import workloads
from tests.gpu_util import need_gpu, np_

pytestmark = pytest.mark.gpu


def _matrix(kind, r, c):
    if kind == "constant":
        return np.where((np.arange(r * c) % 3 == 0), -1.5, 1.5).astype(np.float32).reshape(r, c)
    if kind == "two":   # the quantile falls between two magnitudes
        return np.where((np.arange(r * c) % 100 < 99), 1.0, 64.0).astype(np.float32).reshape(r, c)
    if kind == "sparse":
        x = np.zeros((r, c), np.float32)
        x.reshape(-1)[::97] = np.float32(0.25)
        return x
    return workloads.matrix(r, c, seed=r + c)


@pytest.mark.parametrize("kind", ["t_rows", "constant", "two", "sparse"])
@pytest.mark.parametrize("shape", [(16, 16), (16, 144), (48, 176), (272, 1040), (1040, 272), (528, 4112)])
@pytest.mark.parametrize("q", [0.0, 0.5, 0.99, 1.0])
def test_threshold_of_quantize(kind, shape, q):
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    x = _matrix(kind, *shape)
    wide = torch.zeros((2, shape[0], shape[1] + 16), device="cuda")   # rows not contiguous
    wide[0, :, :shape[1]] = torch.from_numpy(x)
    wide[1, :, :shape[1]] = torch.from_numpy(x) * 2
    tau = clip_threshold(x, np.float32(q))
    for t in (wide[:, :, :shape[1]], wide[:, :, :shape[1]].contiguous()):
        *_, got, _ = F.fp4root_quantize(t, axis=1, flags=F.F_DEFAULT, clip_quantile=q)
        assert np_(got)[0] == tau and np_(got)[1] == np.float32(2) * tau


@pytest.mark.parametrize("kind", ["t_rows", "constant", "two", "sparse"])
@pytest.mark.parametrize("shape", [(16, 16), (48, 176), (1040, 272), (528, 4112)])
def test_clipped_and_normalised(kind, shape):
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    x = _matrix(kind, *shape)
    buf = torch.zeros((shape[0], shape[1] + 16), device="cuda")
    buf[:, :shape[1]] = torch.from_numpy(x)
    out = F.fp4root_orthogonalize([buf[:, :shape[1]]], steps=0)[0]
    ref, tall, _ = ns.prepare(x)
    assert np.array_equal(np_(out), ref.T if tall else ref)


def test_more_matrices_than_a_chunk():
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    mats = [workloads.matrix(*((48, 80) if i % 3 else (80, 48)), seed=i) for i in range(131)]
    ins = [torch.from_numpy(m).cuda() for m in mats]
    outs = F.fp4root_orthogonalize(ins, steps=2)
    co = F.fp4root_default_coeffs(48, 80, 2)
    for i in (0, 1, 127, 128, 129, 130):
        assert np.array_equal(np_(outs[i]), ns.orthogonalize(mats[i], co, seed=0)), i
    for i in range(0, 131, 7):   # every matrix equals a call on it alone
        alone = F.fp4root_orthogonalize([ins[i]], steps=2)[0]
        assert torch.equal(alone, outs[i]), i
