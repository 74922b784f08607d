"""The bunch field solve over the grids where its sine-mode preconditioner can
go wrong (edges of its 64-column, 32-row tiles and of the radial sweeps, the
smallest and the longest radial system, one row more than a sweep's
threads) and the widest grids, which keep the diagonal, against the oracle's
direct solve.

Bars: |phi error| <= cond(K) * residual, and the fields are differences of phi
over a cell.  The residual is 1e-13 and cond(K) at most 3e4 (the systems
scaled to a unit diagonal; 193 x 300 has the largest), so
1e-8 of each field's maximum.
"""
import numpy as np
import pytest

from inputs import bunch_particles
from test_gpu_bunch import E, bunch_mod  # noqa: F401  (fixtures)
from test_gpu_parity import ferr, say, staggered

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,nr,beta,w", [
    (4, 2, 0.9, 1.0), (5, 33, 0.0, 1.0), (17, 31, 0.99, 1.0), (65, 32, 0.99, 1.0), (66, 34, 0.999, 1e-30),
    (97, 65, 0.9, 1e30), (193, 300, 0.9, 1.0), (40, 513, 0.99, 1.0), (6, 1025, 0.9, 1.0), (5, 4094, 0.9, 1.0),
    (16384, 3, 0.9, 1.0), (16400, 4, 0.9, 1.0)])
def test_bunch_solve_grids(E, bunch_mod, nx, nr, beta, w):  # noqa: F811
    cfg = dict(nx=nx, nr=nr, dx=0.8, dr=1.5, dt=0.6, n_modes=1, profile="none", a0=0.0, ppc=(1, 1, 1),
               shape_order=1, capacity=2 * nx * nr + 4000)
    say("bunch solve", nx, nr, beta, w)
    g = E.Sim(cfg, E.FP64)
    g.set_particles(bunch_particles(1000, 12, x0=0.5 * nx * 0.8, sig_x=0.08 * min(nx, 100), sig_r=0.08 * nr * 1.5,
                                    p0=2.0, w_total=w))
    it, res = g.bunch_fields(0, 1000, beta, tol=1e-13)
    say("iterations", it, "residual", res)
    assert 0 < it and res <= 1e-13
    ex, er, bt, _, _ = bunch_mod.bunch_fields(cfg, g.get_particles(), beta)
    for name, ref in (("ex", ex), ("er", er), ("bt", bt), ("bt_bar", bt)):
        e = ferr(staggered(name, g.get_field(name)), ref)
        say("field", name, f"{e:.2e}")
        assert e <= 1e-8, (name, e)
