"""AdamW's square roots and quotients where the quick forms give way to the general ones.

Blocks whose second moment is zero, subnormal, below or above the quick forms' range, whose
quotients are subnormal, and eps outside their bounds, beside ordinary blocks in the same
wave: weights and both states equal the oracle's bit for bit.
"""
import numpy as np
import pytest
import torch

from oracle import qadamw as Q
from oracle.formats import unpack_nibbles
from tests.gpu_util import need_gpu, np_

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("eps", [1e-8, 1e-35, 1e10])
@pytest.mark.parametrize("scales", [(1.0, 0.0), (1.0, 1e-21, 1e-15), (1e-38, 1e-36, 0.0), (1.0, 1e7, 1e-12), (1e13, 1e-3)])
def test_ranges(scales, eps):
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    n, seed = 256 * 65, 3
    rng = np.random.default_rng(len(scales))
    w_np = Q.bf16_round((rng.standard_normal(n) * 0.02).astype(np.float32))
    w = torch.from_numpy(w_np.view(np.int16).copy()).cuda().view(torch.bfloat16)
    st = F.QAdamWState(n, keep_m=True)
    m_prev = v_prev = None
    for t in range(2):
        f = np.array(scales, np.float32)[rng.integers(0, len(scales), n // 16)]
        g_np = (rng.standard_normal(n).astype(np.float32) * np.repeat(f, 16)).astype(np.float32)
        g_np[rng.integers(0, n, 40)] = 0
        F.fp4root_qadamw_update(w, torch.from_numpy(g_np).cuda(), st, t, 1e-3, 0.1, 0.9, 0.95, eps, flags=22, seed=seed)
        w_np, ms, vs, m_t, _ = Q.adamw_step(g_np, w_np, m_prev, v_prev, t, 1e-3, 0.1, 0.9, 0.95, eps, seed,
                                            hadamard=True, adaptive46=True, sr=True)
        m_prev, v_prev = ms, vs
        assert F.fp4root_device_status(st.ws) == 0
        assert np.array_equal(np_(st.m), m_t)
        assert np.array_equal(unpack_nibbles(np_(st.m_codes)), ms.codes.reshape(-1))
        assert np.array_equal(st.v_means.cpu().numpy().view(np.uint16), vs.means)
        assert np.array_equal(st.v_scales.cpu().numpy().view(np.uint16), vs.scales)
        assert np.array_equal(unpack_nibbles(np_(st.v_codes)), vs.codes)
        assert np.array_equal(w.view(torch.int16).cpu().numpy().view(np.uint16), w_np)
