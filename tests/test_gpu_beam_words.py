"""The beam parameters and the conserved sums where their passes go through a
work item in words of 64 particles: items that end inside, at and after a
word, a range that holds all, some or none of them, and work items longer
than the others (a column injected with many particles per cell).

Bars: as in test_gpu_beam.py; the sums of at most 10^5 FP64 terms, in another
order, to 1e-12 of the sum of their magnitudes.
"""
import numpy as np
import pytest

from inputs import beam_particles
from test_gpu_beam import E, beam_mod, check, say  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def check_all(g, beam_mod, queries):  # noqa: F811
    parts = g.get_particles()
    for q in queries:
        out, hist = g.beam(*q, with_hist=True)
        ref, rhist = beam_mod.beam_parameters(parts, *q)
        check(out, hist, ref, rhist)
    d = g.diagnostics()
    n = len(parts["id"])
    p2 = parts["px"]**2 + parts["py"]**2 + parts["pz"]**2
    terms = {"count": np.ones(n), "charge": -parts["w"], "kin": parts["w"] * p2 / (1 + np.sqrt(1 + p2)),
             "px": parts["w"] * parts["px"],
             "lx": parts["w"] * (parts["y"] * parts["pz"] - parts["z"] * parts["py"])}
    size = {k: np.abs(t).sum() for k, t in terms.items()}
    # (y p_z and z p_y nearly cancel where the momentum is radial: rounding goes by their own size)
    size["lx"] = (parts["w"] * (np.abs(parts["y"] * parts["pz"]) + np.abs(parts["z"] * parts["py"]))).sum()
    for k, t in terms.items():
        assert abs(d[k] - t.sum()) <= 1e-12 * size[k], k


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("n_bulk,n_beam", [(0, 1), (1, 62), (0, 64), (30, 35), (400, 113), (100, 5000)])
def test_words_of_small_and_full_items(E, beam_mod, prec, n_bulk, n_beam):  # noqa: F811
    say("words", prec, n_bulk, n_beam)
    cfg = dict(nx=48, nr=20, dx=0.8, dr=1.5, dt=0.6, n_modes=1, profile="none", a0=0.0, ppc=(1, 1, 1),
               capacity=20000)
    g = E.Sim(cfg, E.FP64 if prec == "fp64" else E.FP32_BULK)
    g.set_particles(beam_particles(cfg, n_bulk, n_beam, seed=73))
    check_all(g, beam_mod, [(0.0, 600.0, 4096), (100.0, 600.0, 50), (395.0, 405.0, 3), (1000.0, 2000.0, 8)])


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_words_of_long_injected_items(E, beam_mod, prec):  # noqa: F811
    """256 particles per cell: an injected item holds 4096, beyond the share
    of the other items."""
    say("long items", prec)
    cfg = dict(nx=24, nr=18, dx=0.8, dr=1.5, dt=0.6, n_modes=1, profile="uniform", n0=0.01, ppc=(4, 8, 8),
               a0=3.0, w0=8.0, tau=4.0, x_c=10.0, x_f=10.0, moving_window=1, seed=191204690)
    g = E.Sim(cfg, E.FP64 if prec == "fp64" else E.FP32_BULK)
    g.step(2)
    check_all(g, beam_mod, [(0.0, 20.0, 256), (1e-4, 20.0, 64)])
