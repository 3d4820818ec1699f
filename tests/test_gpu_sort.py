"""The tile sort: storage order of the particles after it, on random and cell-ordered
loads, with tiles that divide the grid or not, one dense cell, and counts that
span several scan blocks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,t1,t2,per,dense", [
    ((64, 32), 16, 8, 3, 0), ((64, 33), 5, 7, 2, 0), ((8, 4), 4096, 4096, 1, 0), ((128, 65), 32, 8, 1, 3000),
    ((256, 200), 1, 1, 1, 0), ((16, 9, 7), 8, 4, 2, 0), ((32, 24, 17), 5, 3, 3, 500), ((64, 40, 40), 8, 4, 1, 0)])
@pytest.mark.parametrize("shuffled", [False, True])
def test_order_after_a_sort(hpic, n, t1, t2, per, dense, shuffled):
    gen = np.random.default_rng(7)
    dim, cells = len(n), int(np.prod(n))
    cell = np.concatenate([np.repeat(np.arange(cells), per), np.full(dense, cells // 3)])
    if shuffled:
        gen.shuffle(cell)
    i = np.stack(np.unravel_index(cell, n[::-1])[::-1])  # x1 fastest
    x = (i + gen.uniform(0.05, 0.95, i.shape)) * 0.2
    kw = dict(n3=n[2], dx3=0.2) if dim == 3 else {}
    sim = hpic.Sim([hpic.config(n[0], n[1], 0.2, 0.2, 0.05, precision="fp32", **kw)])
    sim.set_particles(0, x, gen.normal(0, 0.1, (3, cell.size)), np.ones(cell.size))
    sim.set_tiling(t1, t2, 4)
    raw = sim.particles_raw(0)
    sim.close()
    assert np.array_equal(np.sort(raw["id"]), np.arange(cell.size))
    assert np.array_equal(raw["cell"][:dim], i[:, raw["id"]])  # every particle whole
    # tiles one after the other
    T = np.minimum([t1, t2, t2][:dim], n)
    nt = [-(-m // t) for m, t in zip(n, T)]
    a = raw["cell"][:dim] // T[:, None]
    tile = a[0] + nt[0] * (a[1] + (nt[1] * a[2] if dim == 3 else 0))
    assert np.all(np.diff(tile) >= 0)
    # of a full tile with as many particles in every cell, the first ones lie in
    # different cells
    if not dense:
        area = int(np.prod(T))
        full = np.flatnonzero(np.bincount(tile, minlength=int(np.prod(nt))) == per * area)
        flat = np.ravel_multi_index(tuple(raw["cell"][:dim][::-1]), n[::-1])
        for t in full[:50]:
            assert np.unique(flat[np.flatnonzero(tile == t)[:area]]).size == area


# counts at the edges of the blocks of 256 particles and of their order in eight runs
@pytest.mark.parametrize("np_", [1, 255, 7 * 256, 7 * 256 + 1, 8 * 256, 8 * 256 + 1, 17 * 256 - 1])
def test_every_particle_once_for_any_count(hpic, np_):
    gen = np.random.default_rng(np_)
    i = np.stack([gen.integers(0, 64, np_), gen.integers(0, 30, np_)])
    sim = hpic.Sim([hpic.config(64, 30, 0.2, 0.2, 0.05, precision="fp32")])
    sim.set_particles(0, (i + gen.uniform(0.05, 0.95, i.shape)) * 0.2, gen.normal(0, 0.1, (3, np_)),
                      np.ones(np_))
    sim.set_tiling(8, 4, 4)
    raw = sim.particles_raw(0)
    sim.close()
    assert np.array_equal(np.sort(raw["id"]), np.arange(np_))
    assert np.array_equal(raw["cell"][:2], i[:, raw["id"]])
    a = raw["cell"][:2] // np.array([[8], [4]])
    assert np.all(np.diff(a[0] + 8 * a[1]) >= 0)
