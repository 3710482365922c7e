"""The optimizer step's shared launches against one call per parameter, bit for bit.

More parameters than one launch takes, shapes whose last workgroup is partial, a weight
listed twice (its updates keep their order), both momentum roundings, two steps.
"""
import pytest
import torch

from paper_2607_04422_amd import workloads
from tests.gpu_util import need_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("momentum_flags", [22, 6, 0])
@pytest.mark.parametrize("count,tied", [(1, False), (32, False), (33, True), (70, True)])
def test_against_single_calls(count, tied, momentum_flags):
    need_gpu()
    from paper_2607_04422_amd import fp4root as F
    shapes = [(16, 16), (48, 144), (144, 48), (64, 64), (272, 16)]
    ws, gs = [], []
    for i in range(count):
        r, c = shapes[i % 5]
        ws.append(torch.from_numpy(workloads.matrix(r, c, seed=i)).cuda().to(torch.bfloat16))
        gs.append(torch.from_numpy(workloads.matrix(r, c, seed=1000 + i)).cuda())
    if tied:
        ws[5] = ws[0]
        ws[15] = ws[10]
    memo = {}
    mine = [memo.setdefault(id(w), w.clone()) for w in ws]
    lr, wd, beta, seed = 0.02, 0.1, 0.9, 7
    root = F.RootStep(ws, gs, lr=lr, wd=wd, beta=beta, steps=1, momentum_flags=momentum_flags, momentum_seed=seed)
    states = [F.MomentumState(1, *g.shape) for g in gs]
    for step in range(2):
        root(step)
        assert root.status() == 0
        ms = [F.fp4root_momentum_update(g, st, beta, step, flags=momentum_flags, seed=seed + i)
              for i, (g, st) in enumerate(zip(gs, states))]
        os_ = F.fp4root_orthogonalize(ms, steps=1)
        for w, o in zip(mine, os_):
            F.fp4root_apply_update(w, o, lr, wd, max(1.0, o.shape[0] / o.shape[1]) ** 0.5)
        for i in range(count):
            assert torch.equal(root.states[i].codes, states[i].codes), i
            assert torch.equal(root.states[i].scales, states[i].scales), i
            assert torch.equal(root.states[i].tensor_scale, states[i].tensor_scale), i
            assert torch.equal(root.scratch[i], os_[i]), i
            assert torch.equal(ws[i], mine[i]), i
