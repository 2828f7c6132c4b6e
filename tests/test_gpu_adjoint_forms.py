"""The adjoint passes' two forms (one line per line group, its field and
adjoint state kept in registers between the fused passes; blocks of several
lines) give the same gradient, at the axial sizes where the last workgroup is
partly filled, for every law, domain and z-boundary condition.  They regroup
sums of the same terms: bounds as between chunk shapes (J 1e-12, gradient
1e-11 of its largest normalised component)."""
import numpy as np
import pytest

import cellgen

from gpu_util import say

pytestmark = pytest.mark.gpu


def _cell(kind, nr, nz):
    c = cellgen.tiny(7, nr=nr, nz=nz, n_layers=4, nsteps=12, z_active=True, dt=2e-6,
                     amplitude=4e9, heater=2)
    if kind == "poly":
        c = cellgen.poly_variant(c, 1, joule_tref=30.0)
    elif kind in ("general", "general_stepped"):
        for m, l in enumerate(c["layers"]):
            l["q"] = 2.5 + 0.25 * (m % 3)
    elif kind == "held":
        c["bc"] = [[0, 0.0], [1, 28.0], [1, 29.0], [1, 28.5]]
    elif kind == "held_z":
        c["bc"] = [[0, 0.0], [0, 0.0], [1, 29.0], [1, 28.5]]
    if kind in ("stepped", "general_stepped"):
        c["stepped"] = dict(z_full=max(1, nz // 2), nr_top=max(3, nr // 3))
    return c


def _plan(cell, shape, lpw):
    import paper_1408_5853_amd as P
    plan = P.Plan(cell)
    plan.set_shape(shape[0], shape[1], lpw)
    return plan


@pytest.mark.parametrize("shape", [(2, 1), (8, 1), (4, 2), (8, 4)])
@pytest.mark.parametrize("kind", ["plain", "general", "poly", "held", "held_z",
                                  "stepped", "general_stepped"])
def test_one_line_form_equals_blocks_of_lines(kind, shape):
    import paper_1408_5853_amd as P
    nr = 64 * shape[0] * shape[1] - 11
    if "stepped" in kind and shape == (8, 4):
        # two row-table sets of 2048 rows: more LDS than a workgroup has
        with pytest.raises(P.CryoError):
            _plan(_cell(kind, nr, 10), shape, 1).gradient(np.zeros(12))
        return
    for nz in (4, 5, 10, 11, 18, 27):
        c = _cell(kind, nr, nz)
        say("case adjoint forms %s shape %s nr %d nz %d" % (kind, shape, nr, nz))
        rng = np.random.default_rng([nz, nr])
        T0 = c["T_init"] + rng.uniform(0.0, 1.0, (nz, nr))
        tgt = c["T_init"] + 0.5 * np.arange(12) / 12
        got = []
        for lpw in (1, 2):
            J, g, _ = _plan(c, shape, lpw).gradient(tgt, T0=T0, ckpt=5)
            got.append((J, g))
        assert got[0][0] == pytest.approx(got[1][0], rel=1e-12)
        th = np.abs(P.params_of(c))
        scale = np.max(np.abs(got[1][1] * th))
        e = float(np.max(np.abs(got[0][1] - got[1][1]) * th))
        say("  largest difference %.3e of %.3e" % (e, scale))
        # (a held outer wall leaves nothing to differentiate: both are zero)
        assert e <= 1e-11 * scale
