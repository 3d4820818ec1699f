"""Quasi-3D tiles follow the particles that are loaded: with ten a cell and more they are
half as high where few workgroups would be left, with fewer they are not."""
import numpy as np
import pytest

from test_gpu_q3d_particles import _by_id, _plasma, _random_fields
from test_gpu_warm import _push_us

pytestmark = pytest.mark.gpu


# 992 tiles of 16 x 4 cells; half as high, a push of two a cell took 0.3 of one of 32
@pytest.mark.parametrize("prec,modes", [("fp64", 2), ("fp64", 1)])
def test_sparse_columns_keep_high_tiles(hpic, prec, modes):
    n1, n2, fill, dz, dr = 512, 124, 104, 0.1, 0.2

    def push(ppc):
        gen = np.random.default_rng(15)
        shape = (n1, fill, ppc)
        r = (np.arange(fill)[None, :, None] + gen.random(shape)) * dr
        th = 2 * np.pi * gen.random(shape)
        z = (np.arange(n1)[:, None, None] + gen.random(shape)) * dz
        x = np.stack([v.ravel() for v in (z, r * np.cos(th), r * np.sin(th))])
        u = np.zeros_like(x)
        u[0] = 20.0
        cfg = hpic.config(n1, n2, dz, dr, 0.02, precision=prec, modes=modes)
        return _push_us(hpic, cfg, x, u, (1e-3 / ppc * r).ravel(), 64)
    assert push(2) < 0.25 * push(32)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_reloads_change_the_tiles(hpic, prec):
    """Loads of 2 and 12 particles a cell in turn, and a saved state, into handles that
    held the others: as in a new handle.  (256 x 92 cells are 368 tiles of 16 x 4 for FP64,
    and with four modes 736 of 8 x 4 for FP32.)"""
    n1, n2, M = 256, 92, 2 if prec == "fp64" else 4
    gen = np.random.default_rng(17)
    E, B = (_random_fields(gen, M, n1, n2, 0.01) for _ in range(2))
    loads = [_plasma(gen, n1, n2, 0.2, 0.25, 70, ppc=p, uth=0.1) for p in ((1, 1, 2), (2, 2, 4))]

    def run(sim, k):
        x, u, w = loads[k]
        for m in range(M):
            sim.set_fields_mode(0, m, E[m], B[m])
        sim.set_particles(0, x, u, w)
        sim.step(4)
        return out(sim)

    def out(sim):
        p = _by_id(sim.particles(0))
        return [sim.field_mode(0, c, m) for c in range(6) for m in range(M)] + [p["x"], p["u"]]

    def new():
        return hpic.Sim([hpic.config(n1, n2, 0.2, 0.25, 0.01, precision=prec, modes=M)])
    want, states = [], []
    for k in (0, 1):
        sim = new()
        want.append(run(sim, k))
        states.append(sim.get_state())
        sim.close()

    def same(got, k):
        for a, b in zip(got, want[k]):
            # FP64: another order of the deposit's sums, over 4 steps
            assert np.array_equal(a, b) if prec == "fp32" else np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
    sim = new()
    for k in (0, 1, 0):
        same(run(sim, k), k)
    for k in (1, 0):
        sim.set_state(states[k])
        same(out(sim), k)
    sim.step(2)
    sim.close()
