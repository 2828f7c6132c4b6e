"""Increments far below the largest one of their line.  An FP32 pair at 4 K
holds increments of 2^-46 K; one step heats a layer by tens of kelvins, and
the rows beyond it, where the increment falls by orders of magnitude per chunk,
must come out to that place, whatever the strength of the rows' coupling:
within 2^-46 K and FP32's relative error of the oracle's increment.  Each row
multiplies that by the error of two laws 2^y in float, |y| below 64: 2^-24
times 64 each."""
import numpy as np
import pytest

import cellgen
import oracle

from gpu_util import say

pytestmark = pytest.mark.gpu


def _cell(nr, fall):
    """Three layers, the middle one heated; next to it the increment falls by
    2^-fall per row."""
    c = cellgen.tiny(2, nr=nr, nz=4, n_layers=3, nsteps=1, z_active=False, dt=1e-7, heater=1)
    c.update(T_init=4.0, t_on=0.0, width=1e-7, period=2e-7)
    c["bc"] = [[0, 0.0]] * 4
    n = (nr - 1) // 3
    ints = [n, n, nr - 1 - 2 * n]
    # an implicit row: x_{i+1} / x_i = g with g + 1/g = 2 + s, s the row's
    # capacity over its face coefficient
    g = 2.0 ** -fall
    s = g + 1.0 / g - 2.0
    for l, k in zip(c["layers"], ints):
        l.update(intervals=k, thickness=2e-6 * k, p=1.0, q=2.0)
        cap = l["rho"] * l["c0"] * (4.0 / l["tref"]) ** l["q"] / c["dt"]
        l["k0"] = cap * (2e-6) ** 2 / s / (4.0 / l["tref"]) ** l["p"]
    h = c["layers"][1]
    c["amplitude"] = 32.0 * h["rho"] * h["c0"] * (4.0 / h["tref"]) ** h["q"] / c["dt"]
    c["height"] = 1.0
    return c


def _increments(c):
    """The step's increments on a line of the uniform field: the oracle's rows
    with the source as the only residual (the field itself cancels, which in
    64 bits leaves more than 2^-46 K of a forward solve's result)."""
    T = oracle.initial_field(c)
    A, B, C, F = oracle.line_rows(c, T, 0, 1)
    M = np.diag(B) + np.diag(A[1:], -1) + np.diag(C[:-1], 1)
    n0, n1 = (sum(l["intervals"] for l in c["layers"][:k]) for k in (1, 2))
    res = np.zeros(c["nr"])
    res[n0 + 1:n1] = (F - M @ T[1])[n0 + 1:n1]
    return oracle.thomas(A, B, C, res)


@pytest.mark.parametrize("shape", [(2, 1, 1), (8, 1, 1), (8, 1, 2), (4, 2, 1), (4, 4, 2)])
@pytest.mark.parametrize("per_chunk", [1.0, 6.0, 12.0, 23.0, 30.0, 38.0, 42.0, 46.0])
def test_increments_of_quiet_rows(per_chunk, shape):
    import torch

    import paper_1408_5853_amd as P
    nr = 64 * shape[0] * shape[1]
    c = _cell(nr, per_chunk / shape[0])
    say("case quiet rows shape %s, 2^-%g per chunk" % (shape, per_chunk))
    plan = P.Plan(c, "f32")
    plan.set_shape(*shape)
    T = plan.init()
    plan.forward(T, 0, 1)
    torch.cuda.synchronize()
    x, xo = plan.field_values(T)[1] - 4.0, _increments(c)
    assert 1.0 < xo.max() < 100.0
    worst = np.max(np.abs(x - xo) / (2.0 ** -46 + 128 * nr * 2.0 ** -24 * xo))
    say("  largest increment %.3g, error %.3g of the bound" % (xo.max(), worst))
    assert worst < 1.0
