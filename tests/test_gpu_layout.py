"""The layout conversions around the stepping kernel: a field loaded into a
resident state (or a batch) and stored again comes back bit for bit, for
radial sizes with and without padding, every chunk shape's lane count, and
both field types; values past the line never leak into it."""
import numpy as np
import pytest

import cellgen
from gpu_util import say

pytestmark = pytest.mark.gpu


def _random_field(nz, nr, seed):
    return 28.0 + np.random.default_rng([41, seed]).uniform(0.0, 9.0, (nz, nr))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nr,nz,shape", [(5, 3, (2, 1, 1)), (64, 4, (2, 1, 1)), (65, 129, (3, 1, 2)),
                                         (129, 7, (16, 1, 1)), (640, 5, (10, 1, 1)),
                                         (500, 9, (4, 2, 1)), (1024, 6, (16, 1, 2)),
                                         (1025, 5, (8, 4, 1)), (2048, 3, (8, 4, 1))])
def test_state_round_trip(nr, nz, shape, dtype):
    import torch

    import paper_1408_5853_amd as P
    say("case %dx%d %s %s" % (nr, nz, shape, dtype))
    plan = P.Plan(cellgen.tiny(1, nr=nr, nz=nz, n_layers=2), dtype)
    plan.set_shape(*shape)
    T = plan.field_from(_random_field(nz, nr, nr))
    st = P.State(plan, T)
    out = st.store()
    st.poll()
    assert torch.equal(out, T)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_batch_round_trip(dtype):
    import torch

    import paper_1408_5853_amd as P
    sizes = [(5, 3), (64, 130), (333, 17), (1024, 9), (1500, 4), (70, 257)]
    cells = [cellgen.tiny(1, nr=nr, nz=nz, n_layers=2) for nr, nz in sizes]
    b = P.Batch(cells, dtype)
    T = b.init()
    for i, (nr, nz) in enumerate(sizes):
        b.field(T, i).copy_(P.Plan(cells[i], dtype).field_from(_random_field(nz, nr, i)))
    T0 = T.clone()
    ws = b.workspace()
    b.forward(T, 0, 0, ws)
    b.poll(ws)
    assert torch.equal(T, T0)
