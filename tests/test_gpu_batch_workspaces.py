"""A batch called with one workspace after another on a side stream, with no
wait between the calls: each call's fields are those of a call by itself, bit
for bit (the batch's descriptors and graph belong to the call in flight)."""
import pytest

import cellgen

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsteps", [7, 640])       # single launches; replayed blocks
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_workspaces_in_turn(dtype, nsteps):
    import torch

    import paper_1408_5853_amd as P
    say("case batch workspaces %s, %d steps" % (dtype, nsteps))
    cells = [cellgen.tiny(i, nr=70 + 60 * i, nz=90 + 50 * i, n_layers=3, z_active=True, dt=2e-7,
                          amplitude=5e9) for i in range(4)]
    want = []
    for k in range(3):
        b = P.Batch(cells, dtype)
        T, ws = b.init(), b.workspace()
        b.forward(T, 100 * k, nsteps, ws=ws)
        b.poll(ws)
        want.append(T)
    b = P.Batch(cells, dtype)
    fields = [b.init() for _ in range(3)]
    spaces = [b.workspace() for _ in range(2)]
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    for k in range(3):
        b.forward(fields[k], 100 * k, nsteps, ws=spaces[k % 2], stream=s)
    torch.cuda.synchronize()
    for k in range(3):
        assert torch.equal(fields[k], want[k]), k
