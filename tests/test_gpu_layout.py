"""Tile segments, work items and sorts at the sizes where their split changes,
against the oracle.

Bars: those of the parity tests (FP64 1e-9; FP32 1e-4 on grids, 1e-3 on
momenta)."""
import numpy as np
import pytest

from inputs import random_particles
from test_gpu_parity import compare_fields, compare_particles, say

pytestmark = pytest.mark.gpu
PRECS = [("fp64", 1e-9, 1e-9), ("fp32", 1e-4, 1e-3)]


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1912_04674_amd as E
    E.lib()
    return E


def _clustered(cfg, counts, seed):
    """counts[k] electrons in the k-th 16 x 16-cell tile column of the lowest
    tile row (all of a tile's particles inside it), random momenta."""
    dx, dr = cfg["dx"], cfg["dr"]
    parts = random_particles(cfg, int(sum(counts)), seed, pmax=0.3)
    rng = np.random.default_rng(seed + 1)
    tile = np.repeat(np.arange(len(counts)), counts)
    x = (16 * tile + rng.uniform(1, 15, tile.size)) * dx
    r = rng.uniform(0.2, 15.5, tile.size) * dr
    th = rng.uniform(0, 2 * np.pi, tile.size)
    parts.update(x=x, y=r * np.cos(th), z=r * np.sin(th))
    return parts


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("prec,tf,tp", PRECS)
def test_work_item_split(E, oracle_mod, prec, tf, tp, order):
    """Tiles of one particle, one short of a wavefront, one either side of one
    and of several work items (512 particles each on this grid): the first
    sort orders them by cell, the others move the particles that changed
    tile, the last (step 27) orders them by cell again."""
    counts = [1, 63, 64, 65, 511, 512, 513, 1023, 1025, 1600]
    cfg = dict(nx=176, nr=32, dx=0.8, dr=1.5, dt=0.6, n_modes=2, profile="none", a0=0.0, ppc=(1, 1, 1),
               shape_order=order, capacity=40_000)
    say("work item split", prec, "order", order)
    g = E.Sim(cfg, E.FP64 if prec == "fp64" else E.FP32_BULK)
    r = oracle_mod.OracleSim(cfg)
    parts = _clustered(cfg, counts, 77)
    g.set_particles(parts)
    r.set_particles(parts)
    g.step(30)
    r.step(30)
    assert g.state()[2] == r.state()[2]
    compare_fields(g, r, tf, modes=2, names=("chi", "ex", "er", "bt", "bt_bar", "jx", "jr"))
    compare_particles(g.get_particles(), r.get_particles(), tp, 1e-8 if prec == "fp64" else 1e-3)


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("dx,dr,dt", [(0.8, 1.5, 0.6), (1.0, 10.0, 0.96)])
def test_particles_at_the_left_edge_of_a_moving_window(E, oracle_mod, dx, dr, dt, prec, order):
    """Electrons as fast as the window, in its first columns: between two sorts
    they drift up to three columns out of a tile that the window is leaving,
    whose place goes to a tile entering at the front."""
    cfg = dict(nx=64, nr=24, dx=dx, dr=dr, dt=dt, n_modes=1, profile="none", a0=0.0, ppc=(1, 1, 1),
               shape_order=order, moving_window=1, capacity=40_000)
    rng = np.random.default_rng(3)
    n = 3000
    r, th = rng.uniform(1, 20, n) * dr, rng.uniform(-np.pi, np.pi, n)
    parts = dict(x=rng.uniform(0.01, 2.5, n) * dx, y=r * np.cos(th), z=r * np.sin(th), px=rng.uniform(20, 200, n),
                 py=np.zeros(n), pz=np.zeros(n), w=np.full(n, 1e-12), id=np.arange(n, dtype=np.uint32))
    g = E.Sim(cfg, E.FP64 if prec == "fp64" else E.FP32_BULK)
    o = oracle_mod.OracleSim(cfg)
    g.set_particles(parts)
    o.set_particles(parts)
    for _ in range(12):
        g.step(10)
        o.step(10)
        a, b = g.get_particles(), o.get_particles()
        k = np.argsort(b["id"])
        say("left edge", prec, "order", order, "step", g.state()[:2], len(k))
        # (FP32: one within rounding of a column's edge may leave a step earlier or later)
        both = np.intersect1d(a["id"], b["id"])
        assert len(a["id"]) + len(b["id"]) - 2 * len(both) <= (0 if prec == "fp64" else 3)
        for name, size in (("x", dx), ("y", dr), ("z", dr)):
            d = a[name][np.isin(a["id"], both)] - b[name][k][np.isin(b["id"][k], both)]
            assert np.abs(d).max() <= (1e-10 if prec == "fp64" else 2e-4) * size, name
    assert 1000 < len(both) < n


@pytest.mark.parametrize("prec,tf,tp", PRECS)
@pytest.mark.parametrize("small,base", [(True, 64), (True, 576), (False, 64), (False, 4160)])
def test_riders_at_their_limit(E, oracle_mod, small, base, prec, tf, tp):
    """A tile whose segment is full (a multiple of 64 particles, nearly at rest) gets,
    in one tile sort, as many arrivals as ride with its last work item (256 with
    items of 512 particles, 1024 with items of 4096), one fewer and one more,
    three tiles away from each other; then the passes that go through them."""
    limit = 256 if small else 1024
    cfg = dict(nx=160 if small else 512, nr=32 if small else 128, dx=0.8, dr=1.5, dt=0.6, n_modes=2, profile="none",
               a0=0.0, ppc=(1, 1, 1) if small else (8, 8, 4), capacity=20_000 if small else 17_400_000)
    say("riders", prec, limit, base)
    rng = np.random.default_rng(limit + base)
    x, p = [], []
    for tile, n in ((1, limit - 1), (4, limit), (7, limit + 1)):
        edge = 16 * (tile + 1)
        # 0.71 cells a step: one cell before the edge at the cell sort (step 3),
        # one beyond it at the tile sort (step 6)
        x += [edge - rng.uniform(3.2, 3.3, n), edge + rng.uniform(4, 12, base)]
        p += [np.full(n, 3.0), np.zeros(base)]
    x, p = np.concatenate(x), np.concatenate(p)
    r, th = rng.uniform(1, 15, x.size) * cfg["dr"], rng.uniform(-np.pi, np.pi, x.size)
    py, pz = rng.uniform(-0.05, 0.05, (2, x.size))
    parts = dict(x=x * cfg["dx"], y=r * np.cos(th), z=r * np.sin(th), px=p, py=py, pz=pz,
                 w=np.full(x.size, 1e-7), id=np.arange(x.size, dtype=np.uint32))
    g = E.Sim(cfg, E.FP64 if prec == "fp64" else E.FP32_BULK)
    o = oracle_mod.OracleSim(cfg)
    g.set_particles(parts)
    o.set_particles(parts)
    for steps in (6, 1, 1, 2):  # (up to the sort, the sort, an in-place pass, another and the next sort)
        g.step(steps)
        o.step(steps)
        assert g.state()[2] == x.size
        compare_fields(g, o, tf, modes=2, names=("chi", "ex", "er", "bt", "bt_bar", "jx", "jr"))
    compare_particles(g.get_particles(), o.get_particles(), tp, 1e-8 if prec == "fp64" else 1e-3)
    stats = g.sort_stats()
    assert stats["cell"] == 1 and stats["incremental"] >= 2 and stats["rebuilt"] == 0
