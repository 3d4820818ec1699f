"""The 2D push's tile boxes: literal column strides (tile widths 8, 16, 32, 64),
boxes that outgrow them, tiles wider than half the grid (the tile's frame is
centred on it), and rejected particles.  The FP32 form's integer deposit makes
every setting bit-identical, so each is compared with single-row tiles sorted
every step; the FP64 form agrees to the rounding of its atomics.  The k-space
update's strips, whose length the handle's size decides, give the same bits
too."""
import numpy as np
import pytest

from paper_1502_01376_amd import workloads as W

pytestmark = pytest.mark.gpu


def _workload(n1, n2, sigma):
    return W.drift2d(n1, n2, 0.2, 0.2, 0.1, sub=(2, 2), gamma=8.0, sigma_u=sigma, jitter=True,
                     seed=W.SEED0 + 301, name="boxes")


def _state(sim):
    E, B = sim.fields(0)
    raw = sim.particles_raw(0)
    o = np.argsort(raw["id"])
    return [E, B, sim.current_fixed(0)] + [v[..., o] for _, v in sorted(raw.items())]


@pytest.mark.parametrize("n1,n2,sigma", [(64, 32, 0.5), (16, 9, 0.5), (8, 4, 0.1), (128, 21, 4.0)])
def test_every_tile_width_gives_the_same_bits(hpic, n1, n2, sigma):
    d = _workload(n1, n2, sigma)
    ref = None
    # sorted once in 20 steps, a hot plasma outgrows its tiles' literal strides
    for t1, t2, K in [(3, 1, 1), (8, 8, 20), (16, 4, 20), (32, 8, 7), (64, 16, 20), (n1, n2, 20)]:
        sim = hpic.from_workload(d, "fp32")
        sim.set_tiling(t1, t2, K)
        sim.step(20)
        got = _state(sim)
        sim.close()
        if ref is None:
            ref = got
        for a, b in zip(got, ref):
            assert np.array_equal(a, b), (t1, t2, K)


@pytest.mark.parametrize("t1", [8, 16, 32, 64])
def test_fp64_widths_agree(hpic, t1):
    d = _workload(64, 32, 0.5)
    out = []
    for t in (3, t1):
        sim = hpic.from_workload(d, "fp64")
        sim.set_tiling(t, 5, 6)
        sim.step(6)
        out.append(np.concatenate(sim.fields(0)))
        sim.close()
    # sums of at most a few hundred terms in another order, over 6 steps
    assert np.abs(out[0] - out[1]).max() <= 1e-11 * np.abs(out[0]).max()


@pytest.mark.parametrize("precision,big", [("fp32", 3e38), ("fp64", 1e308)])
@pytest.mark.parametrize("comp", [0, 1, 2])
def test_a_non_finite_push_is_reported(hpic, precision, big, comp):
    """A field that overflows the momentum along one axis: HP_ENUMERIC, and
    the particles stay as they were."""
    d = _workload(64, 32, 0.0)
    E = np.zeros_like(d["E"])
    E[comp] = big
    sim = hpic.from_workload(d, precision)
    sim.set_fields(0, E, d["B"])
    before = sim.particles(0)
    sim.step(1)
    with pytest.raises(hpic.HpError) as err:
        sim.synchronize()
    assert err.value.code == hpic.HP_ENUMERIC
    after = sim.particles(0)
    o, q = np.argsort(before["id"]), np.argsort(after["id"])
    for k in ("x", "u"):
        assert np.array_equal(before[k][:, o], after[k][:, q])
    sim.close()


def test_update_strips_give_the_same_bits(hpic):
    """Strips of 1 and 2 rows (small handles) against 8 (a handle with a large
    run), at row counts that leave partial strips."""
    ds = [W.drift2d(n1, n2, 0.2, 0.2, 0.05, sub=(1, 1), gamma=5.0, sigma_u=0.3, jitter=True,
                    seed=W.SEED0 + 302 + n2, name="strips") for n1, n2 in ((64, 33), (256, 161), (2048, 397))]
    batch = hpic.from_workloads(ds, "fp32")
    batch.step(3)
    for r in (0, 1):
        one = hpic.from_workload(ds[r], "fp32")
        one.step(3)
        for a, b in zip(one.fields(0), batch.fields(r)):
            assert np.array_equal(a, b)
        one.close()
    batch.close()
