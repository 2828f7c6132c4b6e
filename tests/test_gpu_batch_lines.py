"""Default lines per wave of a batch: few lines take blocks of one line, many
take blocks of up to four, and either way each instance's field is that of a
single plan, bit for bit (lines per wave regroup work only)."""
import numpy as np
import pytest

import cellgen

from gpu_util import run_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,nz,lines", [(3, 40, 1), (3, 3, 1), (40, 900, 2), (64, 1100, 4)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_default_lines_per_wave(count, nz, lines, dtype):
    import torch

    import paper_1408_5853_amd as P
    say("case batch lines count=%d nz=%d %s" % (count, nz, dtype))
    cells = [cellgen.tiny(i % 3, nr=70 + 20 * (i % 4), nz=nz, n_layers=3, z_active=True, dt=2e-7,
                          amplitude=5e9) for i in range(count)]
    b = P.Batch(cells, dtype)
    assert all(b.shape(i)[2] == lines for i in range(count))
    T, ws = b.init(), b.workspace()
    b.forward(T, 0, 7, ws=ws)
    b.poll(ws)
    torch.cuda.synchronize()
    for i in (0, 1, count - 1):
        ref, _ = run_gpu(cells[i], 7, dtype=dtype, surf=False)
        assert np.array_equal(P.Plan.field_values(b.field(T, i)), ref), i
