"""Quasi-3D handles of five to eight modes, whose tiles leave the fields out of the LDS, and
of runs with different mode counts, which take the kernels of a general one."""
import numpy as np
import pytest

from test_gpu_q3d_particles import _by_id, _plasma, _random_fields
from test_gpu_warm import _column

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("modes", [5, 6, 8])
def test_many_modes_keep_large_tiles(hpic, prec, modes):
    """A push grows with the modes, not with the halo of ever smaller tiles.  (The step
    suits the curvature of eight modes at the axis.)"""
    few, many = (_column(hpic, prec, m, 1e-3, dt=0.01) for m in (4, modes))
    assert many < 0.45 * modes * few, (few, many)


def test_sort_memory_follows_the_cells(hpic):
    """The order of the particles takes 16 bytes a cell however small the tiles: a handle
    of eight modes holds little more than its fields and currents."""
    import torch
    n1, n2, modes = 1024, 255, 8
    plane = n1 * (n2 + 1)
    arrays = plane * modes * (2 * 6 * 16 + 6 * 8 + 2 * 3 * 16 + 3 * 8)
    before = torch.cuda.mem_get_info()[0]
    sim = hpic.Sim([hpic.config(n1, n2, 0.1, 0.2, 0.01, precision="fp32", modes=modes)])
    used = before - torch.cuda.mem_get_info()[0]
    sim.close()
    assert used < 1.1 * arrays, (used, arrays)


@pytest.mark.parametrize("counts", [(1, 3), (2, 4), (4, 6)])
def test_runs_of_different_mode_counts(hpic, counts):
    """FP32 form: the same bits as in handles of their own."""
    runs = []
    for M in counts:
        gen = np.random.default_rng(20 + M)
        x, u, w = _plasma(gen, 32, 17, 0.2, 0.25, 7, ppc=(2, 2, 2), uth=0.2)
        runs.append((M, x, u, w, *(_random_fields(gen, M, 32, 17, 0.1) for _ in range(2))))

    def handle(rs):
        sim = hpic.Sim([hpic.config(32, 17, 0.2, 0.25, 0.01, alpha=0.5, precision="fp32", modes=r[0]) for r in rs])
        for k, (M, x, u, w, E, B) in enumerate(rs):
            for m in range(M):
                sim.set_fields_mode(k, m, E[m], B[m])
            sim.set_particles(k, x, u, w)
        sim.set_tiling(4, 2, 8)
        sim.step(20)
        out = []
        for k, r in enumerate(rs):
            out.append([sim.field_mode(k, c, m) for c in range(6) for m in range(r[0])])
            p = _by_id(sim.particles(k))
            out[-1] += [p["x"], p["u"]]
        sim.close()
        return out
    for got, r in zip(handle(runs), runs):
        for a, b in zip(got, handle([r])[0]):
            assert np.array_equal(a, b)
