"""The adjoint's running row sums on any memory a kernel can write: a gradient
whose workspace is pinned host memory equals the one on device memory bit for
bit (both forms of the passes, one to four rows of a line per thread), and the
oracle's."""
import numpy as np
import pytest

import cellgen
import oracle

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(2, 1, 1), (2, 1, 3), (8, 2, 1), (8, 4, 1), (8, 4, 2)])
def test_workspace_in_host_memory(shape):
    import torch

    import paper_1408_5853_amd as P
    n = 12
    c = cellgen.tiny(7, nr=100, nz=14, n_layers=4, nsteps=n, z_active=True, dt=2e-6,
                     amplitude=4e9, heater=2)
    tgt = c["T_init"] + 0.5 * np.arange(n) / n
    say("case adjoint sums in host memory, shape", shape)
    td = torch.tensor(tgt, dtype=torch.float64, device="cuda")
    got = []
    for pinned in (False, True):
        plan = P.Plan(c)
        plan.set_shape(*shape)
        plan.set_gradient_store(n)
        b = plan.gradient_workspace_bytes(n)
        ws = torch.empty(b, dtype=torch.uint8, pin_memory=True) if pinned else \
            torch.empty(b, dtype=torch.uint8, device="cuda")
        assert ws.data_ptr() % 256 == 0
        J, g, S, _ = plan.gradient_async(td, plan.init(), ws=ws)
        torch.cuda.synchronize()
        got.append((J.item(), g.cpu().numpy(), S.cpu().numpy()))
    assert got[0][0] == got[1][0]
    assert np.array_equal(got[0][1], got[1][1]) and np.array_equal(got[0][2], got[1][2])
    Jo, go, _ = oracle.gradient(c, tgt)
    th = np.abs(P.params_of(c))
    assert got[0][0] == pytest.approx(Jo, rel=1e-9)
    assert np.max(np.abs(got[0][1] - go) * th) < 1e-8 * np.max(np.abs(go * th))
