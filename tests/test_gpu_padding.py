"""Rows past the end of a line (nr is rarely a multiple of a wave's rows) take
no part in a step, whatever the cell: z-boundaries held far from T_init beside
laws whose axial step is unstable at that temperature (the cell itself is held
down by its walls, or starts warm), and fields loaded far from T_init.  Both
stepping forms, several steps per launch and the adjoint against the oracle
(FP64 1e-10 relative, FP32 pairs 1e-4 K; J 1e-9, gradient 1e-8 of its largest
normalised component, as the tests of the same calls hold them)."""
import numpy as np
import pytest

import cellgen
import oracle

from gpu_util import say

pytestmark = pytest.mark.gpu

NR, NZ, NSTEPS = 100, 34, 40


def _bound(cell, T):
    """dt of the explicit axial half step at temperature T."""
    eta = cell["height"] / (cell["nz"] - 1)
    return min(0.5 * eta * eta * l["rho"] * l["c0"] * (T / l["tref"]) ** l["q"]
               / (l["k0"] * (T / l["tref"]) ** l["p"]) for l in cell["layers"])


def _thin_outer(kind):
    """Walls held at 28 K, a z-boundary at 60 K; the outer layer 20 um thick,
    its diffusivity growing with T and at 0.9 of the bound at 28 K."""
    c = cellgen.tiny(5, nr=NR, nz=NZ, n_layers=4, nsteps=NSTEPS)
    o, T, eta = c["layers"][-1], c["T_init"], c["height"] / (NZ - 1)
    o.update(thickness=20e-6, p=2.5, q=1.0)
    if kind == "poly":
        for l in c["layers"]:
            l["poly_a"] = [float(l["c0"]), 0.0, 0.0, 0.0]
            l["poly_b"] = [0.02 * l["k0"], 0.0, 0.0, 0.0, 0.0]
        lam = 0.9 * eta * eta * o["rho"] * o["c0"] / (2.0 * c["dt"])
        o["poly_b"] = [0.0, 0.0, 0.0, 0.0, float(lam / T ** 4)]
        c.update(poly=True, joule_tref=0.0)
    else:
        cap = o["rho"] * o["c0"] * (T / o["tref"]) ** o["q"]
        o["k0"] = 0.9 * eta * eta * cap / (2.0 * c["dt"]) / (T / o["tref"]) ** o["p"]
    c["bc"] = [[1, T], [1, T], [1, 60.0], [0, 0.0]] if kind == "low" else \
              [[1, T], [1, T], [0, 0.0], [1, 60.0]]
    return c, None


def _warm(kind):
    """T_init 4.2 K (dt at 0.9 of the bound there), the field at 77 K, inner
    wall and a z-boundary held at 77 K, outer wall free."""
    c = cellgen.tiny(3, nr=NR, nz=NZ, n_layers=4, nsteps=NSTEPS)
    c["T_init"] = 4.2
    s = 0.9 * _bound(c, c["T_init"]) / c["dt"]
    for k in ("dt", "width", "period", "t_on"):
        c[k] *= s
    c["amplitude"] = 0.02 * min(l["rho"] * l["c0"] * (77.0 / l["tref"]) ** l["q"]
                                for l in c["layers"]) / c["dt"]
    c["bc"] = [[1, 77.0], [0, 0.0], [0, 0.0], [1, 77.0]]
    if kind == "warm_stepped":
        c["stepped"] = dict(z_full=17, nr_top=60)
    return c, 77.0 + np.random.default_rng(1).uniform(0.0, 1.0, (NZ, NR))


def _case(kind):
    return _warm(kind) if kind.startswith("warm") else _thin_outer(kind)


# several steps a launch; blocks of two lines; one line of two waves
SHAPES = [(2, 1, 1), (2, 1, 2), (4, 2, 1)]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", ["top", "low", "poly", "warm", "warm_stepped"])
def test_forward(kind, shape, dtype):
    import torch

    import paper_1408_5853_amd as P
    c, T0 = _case(kind)
    say("case padding %s shape %s %s" % (kind, shape, dtype))
    plan = P.Plan(c, dtype)
    plan.set_shape(*shape)
    T = plan.init() if T0 is None else plan.field_from(T0)
    ws = plan.workspace(NSTEPS)
    surf = torch.zeros(NSTEPS, dtype=torch.float64, device="cuda")
    plan.forward(T, 0, NSTEPS, ws=ws, surf=surf)
    plan.poll(ws)
    torch.cuda.synchronize()
    Tg, Sg = plan.field_values(T), surf.cpu().numpy()
    To, So = oracle.forward(c, T=T0, nsteps=NSTEPS, surf=True)
    inside = np.ones_like(To, dtype=bool)
    if kind == "warm_stepped":
        inside[c["stepped"]["z_full"] + 1:, c["stepped"]["nr_top"]:] = False
    if dtype == "f64":
        assert np.max(np.abs(Tg - To)[inside] / To[inside]) < 1e-10
        assert np.max(np.abs(Sg - So) / So) < 1e-10
    else:
        assert np.max(np.abs(Tg - To)[inside]) < 1e-4
        assert np.max(np.abs(Sg - So)) < 1e-4


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", ["warm", "warm_stepped"])
def test_gradient(kind, shape):
    import paper_1408_5853_amd as P
    c, T0 = _case(kind)
    say("case padding gradient %s shape %s" % (kind, shape))
    tgt = np.full(NSTEPS, 77.0)
    plan = P.Plan(c)
    plan.set_shape(*shape)
    Jg, gg, _ = plan.gradient(tgt, T0=T0, ckpt=7)
    Jo, go, _ = oracle.gradient(c, tgt, T0=T0, nsteps=NSTEPS)
    assert Jg == pytest.approx(Jo, rel=1e-9)
    th = np.abs(P.params_of(c))
    scale = np.max(np.abs(go * th))
    assert scale > 0.0
    assert np.max(np.abs(gg - go) * th) < 1e-8 * scale


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lines", [1, 2])
def test_batch(lines, dtype):
    import torch

    import paper_1408_5853_amd as P
    kinds = ["top", "low", "poly", "warm"]
    say("case padding batch, %d lines per wave, %s" % (lines, dtype))
    cases = [_case(k) for k in kinds]
    b = P.Batch([c for c, _ in cases], dtype, shapes=[(2, 1, lines)] * len(cases))
    T, ws = b.init(), b.workspace()
    for i, (c, T0) in enumerate(cases):
        if T0 is not None:
            b.field(T, i).copy_(P.Plan(c, dtype).field_from(T0))
    b.forward(T, 0, NSTEPS, ws=ws)
    b.poll(ws)
    torch.cuda.synchronize()
    for i, (c, T0) in enumerate(cases):
        To = oracle.forward(c, T=T0, nsteps=NSTEPS)
        e = np.abs(P.Plan.field_values(b.field(T, i)) - To)
        assert np.max(e / To) < 1e-10 if dtype == "f64" else np.max(e) < 1e-4, kinds[i]
