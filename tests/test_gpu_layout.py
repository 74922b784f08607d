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
