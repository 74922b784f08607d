"""The current filter at the edges of its 32 x 32 tiles, for every number of
passes: random currents through the field stage of a vacuum run, against the
oracle's filter of the same currents.

Bars: 2N + 1 products per direction of values of order one with weights that
add up to one, and the rounding of the input: (4N + 4) units of rounding of
the type, of the largest input.
"""
import numpy as np
import pytest

from inputs import C1, scaled
from test_gpu_parity import E, say  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,nr,passes", [(19, 17, 8), (31, 33, 1), (32, 31, 2), (63, 32, 3), (64, 64, 5), (33, 65, 8)])
def test_filter_at_tile_edges(E, oracle_mod, prec, nx, nr, passes):  # noqa: F811
    say("filter tiles", prec, nx, nr, passes)
    cfg = scaled(C1, nx=nx, nr=nr, n_modes=2, profile="none", a0=0.0, filter_passes=passes)
    g = E.Sim(cfg, E.FP64 if prec == "fp64" else E.FP32_BULK)
    r = oracle_mod.OracleSim(cfg)
    rng = np.random.default_rng(nx)
    inputs = {}
    for name, (imax, jmax) in {"jx": (nx - 1, nr), "jr": (nx, nr - 1), "jx1": (nx - 1, nr), "jr1": (nx, nr - 1),
                               "jt1": (nx, nr)}.items():
        f = rng.standard_normal((nx + 1, nr + 1))
        if name.endswith("1"):
            f = f + 1j * rng.standard_normal(f.shape)
        f[imax + 1:, :] = 0
        f[:, jmax + 1:] = 0
        inputs[name] = f
    g.gather_push(E.MOMENTUM)
    g.envelope_step()
    g.gather_push(E.POSITION)
    for name, f in inputs.items():
        g.set_field(name, f)
        r.set_field(name, f)
    g.field_step()
    r.filter_J()
    eps = np.finfo(np.float64 if prec == "fp64" else np.float32).eps
    for name, f in inputs.items():
        err = np.abs(g.get_field(name) - r.get_field(name)).max()
        say(name, f"{err:.2e}")
        assert err <= (4 * passes + 4) * eps * np.abs(f).max(), (name, err)


def test_filtered_current_of_the_entering_column(E, oracle_mod):  # noqa: F811
    """A window run past one turn of the ring of columns (96 here): the filtered
    current of the column that just entered is zero, not what the ring held.
    Bar: the FP64 path's."""
    cfg = dict(nx=31, nr=19, dx=0.8, dr=1.5, dt=0.6, n_modes=2, ppc=(2, 2, 2), profile="uniform", n0=0.01, a0=2.0,
               w0=10.0, tau=6.0, x_c=16.0, x_f=16.0, moving_window=1, filter_passes=3, seed=191204691)
    g = E.Sim(cfg, E.FP64)
    r = oracle_mod.OracleSim(cfg)
    f = 1e-3 * np.ones((32, 20)) + 0j
    f[0] = f[31] = 0
    f[:, 19] = 0
    for s in (g, r):
        s.set_field("er1", f)
        s.set_field("et1", -1j * f)
    g.step(150)
    r.step(150)
    for _ in range(4):
        say("entering column", g.state()[:2])
        for name in ("jx", "jr", "jx1", "jr1", "jt1"):
            ref = r.get_field(name)
            err, size = float(np.abs(g.get_field(name) - ref).max()), float(np.abs(ref).max())
            assert err <= 1e-9 * size, name
        g.step(1)
        r.step(1)
