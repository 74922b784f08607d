"""Work items of a size taken from a full tile's particles (1024 on this grid,
two items of a tile of 1536, where the particles per compute unit alone give
512): tiles of counts either side of one, two and three items, through cell and
tile sorts, against the oracle.

Bars: those of the parity tests (FP64 1e-9; FP32 1e-4 on grids, 1e-3 on
momenta).
"""
import pytest

from test_gpu_layout import E, PRECS, _clustered  # noqa: F401  (fixture)
from test_gpu_parity import compare_fields, compare_particles, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("prec,tf,tp", PRECS)
def test_items_of_a_full_tile(E, oracle_mod, prec, tf, tp, order):  # noqa: F811
    counts = [1, 511, 513, 1023, 1024, 1025, 1536, 1537, 2047, 2048, 2049, 3073]
    cfg = dict(nx=1088, nr=112, dx=0.8, dr=1.5, dt=0.6, n_modes=2, profile="none", a0=0.0, ppc=(1, 2, 3),
               shape_order=order)
    say("items of a full tile", prec, "order", order)
    g = E.Sim(cfg, E.FP64 if prec == "fp64" else E.FP32_BULK)
    r = oracle_mod.OracleSim(cfg)
    parts = _clustered(cfg, counts, 79)
    g.set_particles(parts)
    r.set_particles(parts)
    g.step(8)
    r.step(8)
    assert g.state()[2] == r.state()[2]
    compare_fields(g, r, tf, modes=2, names=("chi", "ex", "er", "bt", "bt_bar", "jx", "jr"))
    compare_particles(g.get_particles(), r.get_particles(), tp, 1e-8 if prec == "fp64" else 1e-3)
