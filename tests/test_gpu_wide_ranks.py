"""The clip threshold of matrices of 2^32 elements and more: ranks beyond 32 bits, and more
equal elements than a 32-bit count holds."""
import pytest
import torch

from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu

ROWS, COLS = 32784, 131072   # 2^32 + 2^21 elements


@pytest.fixture(scope="module")
def big():
    need_gpu()
    x = torch.empty((ROWS, COLS), device="cuda")
    yield x
    del x
    torch.cuda.empty_cache()


# (value of all elements but the last two rows', value of the last row, quantile): a count
# past 2^32 in one bin, a rank past 2^32, and one that falls between the two values
CASES = [(1.0, 3.0, 0.5), (0.0, 5.0, 1.0), (1.0, 3.0, 0.99), (1.0, 1.0, 0.75)]


def _fill(x, low, high):
    x.fill_(low)
    x[-1].fill_(-high)


@pytest.mark.parametrize("low,high,q", CASES)
def test_threshold(big, low, high, q):
    from paper_2607_04422_amd import fp4root as F
    _fill(big, low, high)
    want = high if q == 1.0 else low
    codes, scales, sg, tau, _ = F.fp4root_quantize(big, axis=1, flags=F.F_CLIP, clip_quantile=q)
    assert float(tau[0]) == want
    out = (codes, scales, sg, torch.full((1,), -1.0, device="cuda"), torch.full((1,), 7, dtype=torch.int32, device="cuda"))
    F.fp4root_quantize_noalloc(big, out, axis=1, flags=F.F_CLIP, clip_quantile=q)
    assert float(out[3][0]) == want and int(out[4][0]) == 0


def test_norm_of_the_clipped_matrix(big):
    from paper_2607_04422_amd import fp4root as F
    _fill(big, 1.0, 3.0)
    out = F.fp4root_orthogonalize([big], steps=0)[0]
    # every element is +-1 after clipping at 1: sums of whole numbers below 2^53, so exact
    inv = torch.tensor(1.0 / ((ROWS * COLS) ** 0.5 + float(torch.tensor(1e-7))), dtype=torch.float64).float()
    assert float(out.min()) == -float(inv) and float(out[:-1].min()) == float(out.max()) == float(inv)
