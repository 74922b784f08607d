"""One position push in vacuum against the oracle, over every form that the
radius and azimuth update takes: steps short against the radius (series in
beta = b/(r + a)), either side of the |beta| = 0.05 line, across and onto the
axis, with nothing but azimuthal or radial motion, and reflections at r_max."""
import numpy as np
import pytest

from test_gpu_parity import by_id, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1912_04674_amd as E
    E.lib()
    return E


def _particles(cfg, n, seed):
    rng = np.random.default_rng(seed)
    dx, dr, nr = cfg["dx"], cfg["dr"], cfg["nr"]
    # radii from 1e-7 cells to r_max, a tenth of them in the last cell
    r = dr * np.exp(rng.uniform(np.log(1e-7), np.log(nr * 0.999), n))
    wall = rng.uniform(size=n) < 0.1
    r[wall] = (nr - rng.uniform(1e-6, 0.8, wall.sum())) * dr
    th = rng.uniform(-np.pi, np.pi, n)
    p = 10.0 ** rng.uniform(-8, 1.5, n)  # up to 0.9995 c
    u = rng.normal(size=(3, n))
    kind = rng.integers(0, 4, n)
    c, s = np.cos(th), np.sin(th)
    u[:, kind == 1] = np.stack([0 * c, c, s])[:, kind == 1] * rng.choice([-1, 1], (kind == 1).sum())  # radial
    u[:, kind == 2] = np.stack([0 * c, -s, c])[:, kind == 2]  # azimuthal
    u /= np.linalg.norm(u, axis=0)
    # a few aimed so that the step ends on the axis or near |beta| = 0.05
    k = np.flatnonzero(kind == 2)[:500]
    v = p / np.sqrt(1 + p * p)
    r[k] = cfg["dt"] * v[k] / 0.05 * rng.uniform(0.999, 1.001, k.size)
    k = np.flatnonzero(kind == 1)[:200]
    r[k] = cfg["dt"] * v[k]
    r = np.minimum(r, 0.9999 * nr * dr)
    return dict(x=rng.uniform(4, cfg["nx"] - 4, n) * dx, y=r * c, z=r * s, px=p * u[0], py=p * u[1], pz=p * u[2],
                w=np.full(n, 1e-9), id=np.arange(n, dtype=np.uint32))


# FP64: a few roundings of the azimuth (4e-16 pi) at up to 24 cells, and of
# the radius; FP32: half an ulp of the azimuth (1.2e-7) twice at up to 24
# cells, and the direction cosines (1e-6) times the step of 0.4 cells
@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-13), ("fp32", 1e-5)])
def test_push_all_forms(E, oracle_mod, prec, tol, order):
    cfg = dict(nx=64, nr=24, dx=0.8, dr=1.5, dt=0.6, n_modes=2, profile="none", a0=0.0, ppc=(1, 1, 1),
               shape_order=order, capacity=60_000)
    _push_and_compare(E, oracle_mod, cfg, _particles(cfg, 20_000, 5), prec, tol)


def _push_and_compare(E, oracle_mod, cfg, parts, prec, tol):
    g = E.Sim(cfg, E.FP64 if prec == "fp64" else E.FP32_BULK)
    r = oracle_mod.OracleSim(cfg)
    g.set_particles(parts)
    r.set_particles(parts)
    g.step(1)
    r.step(1)
    a, b = by_id(g.get_particles()), by_id(r.get_particles())
    assert np.array_equal(a["id"], b["id"])
    err = {k: float(np.abs(a[k] - b[k]).max() / cfg[s]) for k, s in (("x", "dx"), ("y", "dr"), ("z", "dr"))}
    say("push", prec, "order", cfg["shape_order"], err)
    assert max(err.values()) <= tol
    # the currents follow the same move (mode 1 at its mid-point)
    for n in ("jx", "jr", "jx1", "jr1", "jt1"):
        ref = r.get_field(n)
        e = float(np.abs(g.get_field(n) - ref).max() / np.abs(ref).max())
        say(n, f"{e:.1e}")
        assert e <= (1e-12 if prec == "fp64" else 2e-5), (n, e)


# The largest moves that the stability limit accepts: with dx well above dr a
# step crosses up to 0.965 dr, so a particle near the top of its cell ends up to
# 1.965 cells above the cell's bottom.  Bars as above (the step is 0.96 cells).
@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-13), ("fp32", 1e-5)])
@pytest.mark.parametrize("dx,dt", [(10.0, 0.96), (3.0, 0.91)])
def test_push_near_the_step_limit(E, oracle_mod, dx, dt, prec, tol, order):
    cfg = dict(nx=64, nr=24, dx=dx, dr=1.0, dt=dt, n_modes=2, profile="none", a0=0.0, ppc=(1, 1, 1),
               shape_order=order, capacity=60_000)
    parts = _particles(cfg, 20_000, 6)
    rng = np.random.default_rng(7)
    # half of them fast and radial, near the top of a cell or anywhere in it,
    # outward (one in four inward)
    k = np.arange(0, 20_000, 2)
    n = k.size
    fr = np.where(rng.uniform(size=n) < 0.5, 1 - 10.0 ** rng.uniform(-6, -1, n), rng.uniform(0, 1, n))
    r = rng.integers(0, cfg["nr"], n) + np.minimum(fr, 0.999999)
    th, p = rng.uniform(-np.pi, np.pi, n), 10.0 ** rng.uniform(0.5, 2, n) * rng.choice([1, 1, 1, -1], n)
    slope = rng.normal(size=(2, n)) * 0.05
    c, s = np.cos(th), np.sin(th)
    for name, v in (("y", r * c), ("z", r * s), ("px", p * slope[0]), ("py", p * (c - s * slope[1])),
                    ("pz", p * (s + c * slope[1]))):
        parts[name][k] = v
    _push_and_compare(E, oracle_mod, cfg, parts, prec, tol)


def test_squares_beyond_fp64(E, oracle_mod):
    """Momenta and magnetic fields that are accepted but whose squares are not
    finite in FP64: 1/gamma and the rotation are zero, as in the oracle (equal
    momenta; the particles at rest, the rest of the bars as above)."""
    cfg = dict(nx=32, nr=16, dx=0.8, dr=1.5, dt=0.6, n_modes=2, profile="none", a0=0.0, ppc=(1, 1, 1))
    parts = dict(x=np.array([8.0, 9, 10, 11]), y=np.array([3.0, 0, 5, 2]), z=np.array([1.0, 4, 0, 2]),
                 px=np.array([1e160, 0.2, 1, 0.1]), py=np.array([0.0, -1e200, 1, 0.2]),
                 pz=np.array([0.5, 1e158, 1, 0.3]), w=np.full(4, 1e-9), id=np.arange(4, dtype=np.uint32))
    for field in (0.0, 1e160):
        say("squares beyond fp64", field)
        g = E.Sim(cfg, E.FP64)
        r = oracle_mod.OracleSim(cfg)
        g.set_particles(parts)
        r.set_particles(parts)
        bt = np.full((cfg["nx"] + 1, cfg["nr"] + 1), field)
        g.set_field("bt_bar", bt)
        r.set_field("bt_bar", bt)
        g.gather_push(E.MOMENTUM)
        r.momentum_chi()
        a, b = by_id(g.get_particles()), by_id(r.get_particles())
        for k in ("px", "py", "pz"):
            np.testing.assert_allclose(a[k], b[k], rtol=1e-13, err_msg=k)
        g.envelope_step()
        r.envelope()
        g.gather_push(E.POSITION)
        r.position_J()
        a, b = by_id(g.get_particles()), by_id(r.get_particles())
        for k in ("x", "y", "z"):
            np.testing.assert_allclose(a[k], b[k], rtol=1e-13, atol=1e-13, err_msg=k)
        g.field_step()
