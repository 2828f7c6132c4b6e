"""Several steps in one launch (grids that leave compute units idle) against
one step per launch: field and surface trace equal bit for bit, at axial sizes
around a workgroup's owned lines, every law, domain and z-boundary condition,
and step counts that leave remainders.  The runs of single steps are the form
that the other tests hold to the oracle; one run of each kind is held to it
here too (FP64 1e-10 relative, FP32 pairs 1e-4 K)."""
import numpy as np
import pytest

import cellgen
import oracle

from gpu_util import say

pytestmark = pytest.mark.gpu

NSTEPS = 11                      # launches of 4, 4, 3 | 3, 3, 3, 2 | 2, 2, 2, 2, 2, 1 steps


def _cell(kind, nr, nz):
    c = cellgen.tiny(5, nr=nr, nz=nz, n_layers=min(4, (nr - 1) // 2), z_active=True,
                     nsteps=NSTEPS, dt=2e-7, amplitude=5e9)
    if kind == "poly":
        c = cellgen.poly_variant(c, 1, joule_tref=30.0)
    elif kind == "general":
        for m, l in enumerate(c["layers"]):
            l["q"] = 2.5 + 0.25 * (m % 3)
    elif kind == "stepped":
        c["stepped"] = dict(z_full=max(1, nz // 2), nr_top=max(3, nr // 3))
    elif kind == "held":
        c["bc"] = [[1, 29.0], [1, 28.0], [1, 30.0], [1, 27.0]]
    elif kind == "held_top":
        c["bc"] = [[0, 0.0], [1, 28.0], [0, 0.0], [1, 31.0]]
    elif kind == "turn_on":
        dt = c["dt"]
        c.update(t_on=3 * dt, period=5 * dt, width=2.6 * dt, turn_on=True)
    return c


def _field(cell):
    rng = np.random.default_rng([17, cell["nr"], cell["nz"]])
    return cell["T_init"] + rng.uniform(0.0, 4.0, (cell["nz"], cell["nr"]))


def _run(cell, dtype, shape, per_call):
    import torch

    import paper_1408_5853_amd as P
    plan = P.Plan(cell, dtype)
    plan.set_shape(*shape)
    T = plan.field_from(_field(cell))
    ws = plan.workspace(NSTEPS)
    surf = torch.zeros(NSTEPS, dtype=torch.float64, device="cuda")
    for k in range(0, NSTEPS, per_call):
        n = min(per_call, NSTEPS - k)
        plan.forward(T, k, n, ws=ws, surf=surf[k:k + n])
        plan.poll(ws)
    torch.cuda.synchronize()
    return plan.field_values(T), surf.cpu().numpy()


CASES = [("plain", 128, nz) for nz in (3, 4, 5, 6, 7, 9, 10, 17, 514, 516, 1026, 1540)]
CASES += [(k, 100, nz) for k in ("poly", "general", "stepped", "held", "held_top", "turn_on")
          for nz in (3, 6, 13, 530)]
CASES += [("plain", nr, 19) for nr in (5, 190, 257, 333, 380, 448, 511, 637)]
CASES += [("stepped", 600, 1100), ("general", 640, 700)]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("kind,nr,nz", CASES)
def test_steps_of_one_launch_equal_single_steps(kind, nr, nz, dtype):
    rpl = next(r for r in (2, 3, 4, 5, 6, 7, 8, 10) if 64 * r >= nr)
    say("case %s nr=%d nz=%d %s rpl %d" % (kind, nr, nz, dtype, rpl))
    c = _cell(kind, nr, nz)
    T1, S1 = _run(c, dtype, (rpl, 1, 1), 1)
    Tk, Sk = _run(c, dtype, (rpl, 1, 1), NSTEPS)
    assert np.array_equal(Tk, T1)
    assert np.array_equal(Sk, S1)
    Ts, Ss = _run(c, dtype, (rpl, 1, 1), 5)
    assert np.array_equal(Ts, T1) and np.array_equal(Ss, S1)
    if nz > 60:
        return
    To, So = oracle.forward(c, _field(c), nsteps=NSTEPS, surf=True)
    if dtype == "f64":
        e = max(np.max(np.abs(Tk - To) / To), np.max(np.abs(Sk - So) / So))
        say("  max rel err %.3e" % e)
        assert e < 1e-10
    else:
        e = max(np.max(np.abs(Tk - To)), np.max(np.abs(Sk - So)))
        say("  max abs err %.3e K" % e)
        assert e < 1e-4


@pytest.mark.parametrize("dtype,nz", [("f64", 34), ("f64", 1100), ("f32", 1602), ("f32", 2050)])
def test_trace_over_several_surface_reductions(dtype, nz):
    """More steps than one reduction of the surface sums covers, and FP32
    grids of two workgroups per unit."""
    import torch

    import paper_1408_5853_amd as P
    n = 131
    c = _cell("plain", 100, nz)
    say("case surface reductions nz=%d %s" % (nz, dtype))
    got = []
    for per_call in (1, n):
        plan = P.Plan(c, dtype)
        s = P.State(plan, plan.field_from(_field(c)))
        surf = torch.zeros(n, dtype=torch.float64, device="cuda")
        for k in range(0, n, per_call):
            s.forward(k, per_call, surf=surf[k:k + per_call])
        torch.cuda.synchronize()
        got.append((plan.field_values(s.store()), surf.cpu().numpy()))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("kind,nz,n", [("plain", 34, 4), ("plain", 34, 10), ("plain", 1100, 6),
                                       ("plain", 1100, 8), ("turn_on", 1100, 7)])
def test_captured_state_steps_replay(kind, nz, n):
    """An even number of buffer changes on a resident state (a step is one, the
    turn-on model's pulse start 100), captured once and replayed: every replay
    goes on from the last one's result."""
    import torch

    import paper_1408_5853_amd as P
    say("case captured state steps %s nz=%d n=%d" % (kind, nz, n))
    c = _cell(kind, 100, nz)
    plan = P.Plan(c)
    T0 = plan.field_from(_field(c))
    eager, s = P.State(plan, T0), P.State(plan, T0)
    eager.forward(0, n)
    eager.load(T0)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        s.forward(0, n, stream=stream)
    for rep in range(3):
        g.replay()
        eager.forward(0, n)
        torch.cuda.synchronize()
        assert torch.equal(s.store(), eager.store()), rep
