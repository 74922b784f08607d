"""get_particles, get_field and the checkpoint's columns, which the device
packs: every way the ids can lie (dense, with gaps, at both ends of 32 bits,
too sparse for a bitmap, repeated, none, one), both precisions, against the
values set and against the host's ordering of the same particles, which runs
within a step.

Bars: what is only widened or multiplied once is equal; y and z differ by the
rounding of two sine and cosine implementations, 2 ulp each of r.
"""
import numpy as np
import pytest

from test_gpu_parity import say

pytestmark = pytest.mark.gpu

NX, NR, DX, DR = 40, 19, 0.7, 1.1


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1912_04674_amd as E
    E.lib()
    return E


def ids_of(kind, n, rng):
    if kind == "dense":
        return rng.permutation(n)
    if kind == "gaps":
        return 1000 + rng.choice(3 * n, n, replace=False)
    if kind == "ends":
        return np.concatenate([rng.permutation(n - n // 2), 2**32 - 1 - rng.permutation(n // 2)])
    if kind == "high":
        return 2**32 - 1 - rng.permutation(n)
    return rng.integers(0, max(1, n // 2), n)  # repeated


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("kind,n", [("dense", 0), ("dense", 1), ("dense", 33), ("gaps", 4097), ("ends", 5000),
                                    ("high", 5000), ("repeated", 300), ("dense", 20000)])
def test_export_matches_what_was_set(E, prec, kind, n):
    say("export", prec, kind, n)
    cfg = dict(nx=NX, nr=NR, dx=DX, dr=DR, dt=0.5, n_modes=1, profile="none", a0=0.0, ppc=(1, 1, 1),
               capacity=40000)
    g = E.Sim(cfg, E.FP64 if prec == "fp64" else E.FP32_BULK)
    rng = np.random.default_rng(n)
    r, th = NR * DR * np.sqrt(rng.random(n)) * 0.999, rng.uniform(-np.pi, np.pi, n)
    parts = dict(x=rng.random(n) * NX * DX, y=r * np.cos(th), z=r * np.sin(th), px=rng.normal(size=n),
                 py=rng.normal(size=n), pz=rng.normal(size=n), w=rng.random(n),
                 id=ids_of(kind, n, rng).astype(np.uint32))
    g.set_particles(parts)
    real = np.float64 if prec == "fp64" else np.float32
    got = g.get_particles()
    blob = g.save()
    assert len(got["id"]) == n
    np.testing.assert_array_equal(got["id"], np.sort(parts["id"]))
    if kind != "repeated":
        o = np.argsort(parts["id"])
        for k in ("px", "py", "pz", "w"):
            np.testing.assert_array_equal(got[k], parts[k][o].astype(real).astype(np.float64))
        eps = np.finfo(real).eps
        for k, size in (("x", NX * DX), ("y", 4 * NR * DR), ("z", 4 * NR * DR)):  # (azimuth of up to pi, rounded)
            assert n == 0 or np.abs(got[k] - parts[k][o]).max() <= eps * size, k
    h = E.Sim(cfg, E.FP64 if prec == "fp64" else E.FP32_BULK)
    h.load(blob)
    back = h.get_particles()
    np.testing.assert_array_equal(back["id"], got["id"])
    if kind != "repeated":
        np.testing.assert_array_equal(back["w"], got["w"])
    for name in ("env", "ex", "bt"):
        np.testing.assert_array_equal(h.get_field(name), g.get_field(name))
    g.momentum()  # positions, weights and ids as they were
    host = g.get_particles()
    np.testing.assert_array_equal(host["id"], got["id"])
    if kind != "repeated":
        for k in ("x", "w"):
            np.testing.assert_array_equal(host[k], got[k])
        for k in ("y", "z"):
            assert n == 0 or np.abs(host[k] - got[k]).max() <= 4 * 2.3e-16 * NR * DR
    g.envelope_step()
    g.position()
    g.field_step()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,nr", [(4, 2), (5, 3), (33, 17)])
def test_fields_come_back_as_set(E, prec, nx, nr):
    cfg = dict(nx=nx, nr=nr, dx=0.8, dr=1.5, dt=0.5, n_modes=2, profile="none", a0=0.0, ppc=(1, 1, 1),
               capacity=4000)
    say("fields", prec, nx, nr)
    g = E.Sim(cfg, E.FP64 if prec == "fp64" else E.FP32_BULK)
    rng = np.random.default_rng(nx)
    real = np.float64 if prec == "fp64" else np.float32
    dual_x = ("ex", "bt", "br1", "bt1")
    dual_r = ("er", "bt", "er1", "bx1", "bt1")
    for name in ("env", "env_prev", "ex", "er", "bt", "er1", "bx1", "br1", "bt1"):
        a = rng.normal(size=(nx + 1, nr + 1))
        if name in ("env", "env_prev") or name.endswith("1"):
            a = a + 1j * rng.normal(size=a.shape)
        g.set_field(name, a)
        want = a.copy()
        if real == np.float32:
            want = a.astype(np.complex64 if np.iscomplexobj(a) else np.float32).astype(a.dtype)
        if name in ("env", "env_prev"):
            want[:, :2] = a[:, :2]  # FP64 rows
        if name in dual_x:
            want[nx] = 0
        if name in dual_r:
            want[:, nr] = 0
        np.testing.assert_array_equal(g.get_field(name), want)


def test_two_threads_read_one_simulation(E):
    """Reads of one simulation from two threads at once: the particles are
    ordered and the fields packed in scratch memory that the two share."""
    import threading
    cfg = dict(nx=256, nr=48, dx=0.8, dr=1.5, dt=0.6, n_modes=2, profile="uniform", n0=0.002, a0=1.0, w0=20.0,
               tau=20.0, x_c=100.0, x_f=100.0, ppc=(2, 2, 2))
    g = E.Sim(cfg, E.FP32_BULK)
    g.step(4)
    parts, fields = g.get_particles(), {n: g.get_field(n) for n in ("env", "ex", "bt1")}
    blob = bytes(g.save())
    wrong = []

    def read(first):
        for k in range(first, first + 12):
            if k % 3 == 0:
                got = g.get_particles()
                wrong.extend(n for n in parts if not np.array_equal(got[n], parts[n]))
            elif k % 3 == 1:
                wrong.extend(n for n in fields if not np.array_equal(g.get_field(n), fields[n]))
            elif bytes(g.save()) != blob:
                wrong.append("save")

    threads = [threading.Thread(target=read, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong
