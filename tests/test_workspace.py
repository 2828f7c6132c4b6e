"""Workspace sizes: two internal fields and the surface mean's partial sums.
FP32 pairs default to one line per wave; their workspace stays that of blocks
balanced over the compute units, so that large grids still fit the array of
cryo_forward_noalloc, and the traces of many steps come out whole."""
import numpy as np
import pytest

import cellgen
import paper_1408_5853_amd as P

from gpu_util import say


def _expected(nr, nz):
    """Bytes of a default plan of one wave per line (8 lines per workgroup)."""
    rows = 64 * next(r for r in (2, 3, 4, 5, 6, 7, 8, 10, 12, 16) if 64 * r >= nr)
    up = lambda b: (b + 255) // 256 * 256
    lines = min(8, max(1, round((nz - 2) / 2048)))
    groups = -(-(-(-(nz - 2) // lines)) // 8)
    return 256 + 2 * up(8 * nz * rows) + up(8 * 1024 * groups)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nr,nz", [(64, 128), (128, 30000), (256, 16000), (512, 4098),
                                   (512, 8194), (640, 7000), (1024, 4096)])
def test_bytes_of_a_default_plan(nr, nz, dtype):
    c = cellgen.tiny(1, nr=nr, nz=nz, n_layers=3, dt=1e-9)
    assert P.Plan(c, dtype).workspace_bytes(100) == _expected(nr, nz)


@pytest.mark.gpu
@pytest.mark.parametrize("nr,nz", [(512, 8194), (128, 30000)])
def test_large_fp32_grid_without_allocation(nr, nz):
    """300 steps: more than the partial sums of one reduction."""
    import torch
    n = 300
    say("case noalloc f32 %dx%d" % (nr, nz))
    c = cellgen.tiny(1, nr=nr, nz=nz, n_layers=3, dt=1e-9)
    plan = P.Plan(c, "f32")
    T, S = plan.init(), torch.zeros(n, dtype=torch.float64, device="cuda")
    ws = plan.workspace(n)
    for k in range(n):                              # one reduction per step
        plan.forward(T, k, 1, ws=ws, surf=S[k:k + 1])
    plan.poll(ws)
    T2, S2 = plan.init(), torch.zeros(n, dtype=torch.float64, device="cuda")
    plan.forward_noalloc(T2, 0, n, surf=S2)
    torch.cuda.synchronize()
    assert torch.equal(T, T2) and torch.equal(S, S2)
    assert np.all(S2.cpu().numpy() > 0.0)
