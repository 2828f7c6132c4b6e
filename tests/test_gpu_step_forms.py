"""The stepping kernel's two forms (one line per line group with shared axial
faces, and blocks of several lines) at the sizes where they can go wrong:
partly filled workgroups and blocks, several interfaces in one lane's chunk,
chunks that start at an interface, and every law and domain.  Each form
against the oracle (FP64 1e-10 relative, FP32 pairs 1e-4 K), and against each
other bit for bit: they do the same arithmetic.

Radially fine cells, whose couplings need every pass of the cyclic reduction,
have badly conditioned rows: their bound is the solves' unit roundoff times
the rows' condition number."""
import numpy as np
import pytest

import cellgen
import oracle

from gpu_util import say

pytestmark = pytest.mark.gpu


def _field(cell, seed=0):
    """T_init with a smooth bump and seeded noise, warmer than T_init."""
    rng = np.random.default_rng([31, seed])
    z = np.linspace(0.0, 1.0, cell["nz"])[:, None]
    x = np.linspace(0.0, 1.0, cell["nr"])[None, :]
    return cell["T_init"] + 6.0 * np.exp(-8 * (x - 0.6) ** 2) * (1 + 0.3 * np.cos(5 * z)) \
        + rng.uniform(0.0, 0.5, (cell["nz"], cell["nr"]))


def _cell(kind, nr, nz, layers):
    c = cellgen.tiny(3, nr=nr, nz=nz, n_layers=layers, z_active=True)
    if kind == "poly":
        c = cellgen.poly_variant(c, 1, joule_tref=30.0)
    elif kind == "general":
        for m, l in enumerate(c["layers"]):
            l["q"] = 2.5 + 0.25 * (m % 3)
    elif kind == "stepped":
        c["stepped"] = dict(z_full=max(1, nz // 2), nr_top=max(3, nr // 3))
    elif kind == "strong":                # a fine grid: couplings hardly fall off
        for l in c["layers"]:
            l["thickness"] *= 1e-2
    return c


def _run(cell, dtype, shape, n):
    import torch

    import paper_1408_5853_amd as P
    plan = P.Plan(cell, dtype)
    plan.set_shape(*shape)
    T = plan.field_from(_field(cell))
    ws = plan.workspace(n)
    surf = torch.zeros(n, dtype=torch.float64, device="cuda")
    plan.forward(T, 0, n, ws=ws, surf=surf)
    plan.poll(ws)
    torch.cuda.synchronize()
    return plan.field_values(T), surf.cpu().numpy()


CASES = [(kind, nr, nz, layers, rw)
         for kind, nr, nz, layers, rw in [
             ("cube", 60, 3, 12, (16, 1)),       # one line; three interfaces in a chunk
             ("cube", 128, 10, 4, (2, 1)),       # a full workgroup and a line more
             ("cube", 129, 9, 8, (3, 1)),        # one row in the last chunk
             ("cube", 300, 19, 5, (8, 1)),
             ("cube", 640, 11, 9, (10, 1)),
             ("cube", 700, 12, 6, (4, 4)),
             ("cube", 1030, 7, 7, (8, 4)),
             ("cube", 500, 13, 6, (4, 2)),
             ("general", 257, 18, 6, (5, 1)),
             ("general", 1024, 6, 8, (16, 1)),
             ("poly", 200, 17, 7, (4, 1)),
             ("poly", 900, 5, 5, (8, 2)),
             ("stepped", 150, 21, 5, (3, 1)),
             ("stepped", 1020, 10, 6, (16, 1)),
             ("stepped", 400, 12, 9, (4, 2)),
         ]]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("kind,nr,nz,layers,rw", CASES)
def test_forms_agree(kind, nr, nz, layers, rw, dtype):
    n = 6
    cell = _cell(kind, nr, nz, layers)
    say("case %s %dx%d, %d layers, rows and waves %s, %s" % (kind, nr, nz, layers, rw, dtype))
    T1, S1 = _run(cell, dtype, (*rw, 1), n)
    To, So = oracle.forward(cell, T=_field(cell), nsteps=n, surf=True)
    inside = np.ones_like(To, dtype=bool)
    if kind == "stepped":                 # nodes outside the domain are not solved
        inside[cell["stepped"]["z_full"] + 1:, cell["stepped"]["nr_top"]:] = False
    if dtype == "f64":
        assert np.max(np.abs(T1 - To)[inside] / To[inside]) < 1e-10
        assert np.max(np.abs(S1 - So) / So) < 1e-10
    else:
        assert np.max(np.abs(T1 - To)[inside]) < 1e-4
        assert np.max(np.abs(S1 - So)) < 1e-4
    for lpw in (2, 3):
        if lpw > nz - 2:
            continue
        T2, S2 = _run(cell, dtype, (*rw, lpw), n)
        assert np.array_equal(T1[inside], T2[inside]), lpw
        # (the partial sums of the surface mean are grouped by workgroup)
        assert np.max(np.abs(S1 - S2) / S1) < 1e-14


def _condition(cell, T):
    """Largest infinity-norm condition number of the lines' rows, each row
    divided by its diagonal (the rows of the first step)."""
    worst = 0.0
    for j in range(1, cell["nz"] - 1):
        A, B, C, _ = oracle.line_rows(cell, T, 0, j)
        M = np.eye(cell["nr"]) + np.diag((A / B)[1:], -1) + np.diag((C / B)[:-1], 1)
        worst = max(worst, np.abs(M).sum(1).max() * np.abs(np.linalg.inv(M)).sum(1).max())
    return worst


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nr,nz,rw", [(64, 12, (2, 1)), (512, 5, (8, 1)), (1000, 4, (4, 4))])
def test_couplings_that_hardly_fall_off(nr, nz, rw, dtype):
    n = 6
    cell = _cell("strong", nr, nz, 4)
    T0 = _field(cell)
    say("case strong %dx%d, rows and waves %s, %s" % (nr, nz, rw, dtype))
    T, _ = _run(cell, dtype, (*rw, 1), n)
    To = oracle.forward(cell, T=T0, nsteps=n)
    # a solve's error: unit roundoff (FP64: that of the reciprocals, 2.2e-15)
    # times the condition number, of the largest increment; n of them
    u = 2.2e-15 if dtype == "f64" else 2.0 ** -24
    assert np.max(np.abs(T - To)) < n * u * _condition(cell, T0) * np.max(np.abs(To - T0))
