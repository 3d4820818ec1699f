"""The 3D push's two passes: tiles joined or shared out, boxes that outgrow the LDS or
wrap around the grid, tiles of more particles than one round of passes takes, and
rejected particles.  The FP32 form's integer deposit makes every setting
bit-identical; the FP64 form agrees to the rounding of its atomics."""
import numpy as np
import pytest

from paper_1502_01376_amd import workloads as W

pytestmark = pytest.mark.gpu


def _workload(n, sigma, sub=(2, 1, 1), gamma=3.0):
    return W.drift3d(*n, spread=0.05, sigma_u=sigma, gamma=gamma, jitter=True, sub=sub,
                     seed=W.SEED0 + 501, name="boxes3")


def _state(sim):
    E, B = sim.fields(0)
    raw = sim.particles_raw(0)
    o = np.argsort(raw["id"])
    return [E, B, sim.current_fixed(0)] + [v[..., o] for _, v in sorted(raw.items())]


# 256 x 64 x 40 has 1280 tiles of 8 x 8 x 8, which tiles of 8 x 4 x 4 are joined
# to; a dense 16 x 4 x 4 has 19200 particles in the tile of 8 x 4 x 4, more than 32
# rounds of 256 threads
@pytest.mark.parametrize("n,sigma,sub,interp", [
    ((32, 9, 7), 0.5, (2, 1, 1), 0), ((8, 4, 4), 0.3, (2, 2, 1), 1), ((128, 21, 19), 4.0, (1, 1, 1), 0),
    ((16, 4, 4), 0.2, (6, 5, 5), 0), ((256, 64, 40), 0.3, (1, 1, 1), 1)])
def test_every_tile_gives_the_same_bits(hpic, n, sigma, sub, interp):
    d = _workload(n, sigma, sub)
    ref = None
    # sorted once in 12 steps, a hot plasma outgrows its tiles' boxes
    for t1, t2, K in [(5, 3, 1), (8, 4, 12), (8, 8, 5), (16, 4, 12), (4, 2, 12), (n[0], n[1], 12)]:
        sim = hpic.from_workload(d, "fp32", interp=interp)
        sim.set_tiling(t1, t2, K)
        assert tuple(sim.tiling()["tile"]) == (t1, t2)
        sim.step(12)
        got = _state(sim)
        sim.close()
        ref = ref or got
        for a, b in zip(got, ref):
            assert np.array_equal(a, b), (t1, t2, K)


@pytest.mark.parametrize("n", [(32, 9, 7), (256, 64, 40)])
def test_fp64_tiles_agree(hpic, n):
    d = _workload(n, 0.5)
    out = []
    for t1, t2 in ((3, 2), (8, 4), (8, 8)):
        sim = hpic.from_workload(d, "fp64")
        sim.set_tiling(t1, t2, 6)
        sim.step(6)
        out.append(np.concatenate(sim.fields(0)))
        sim.close()
    for o in out[1:]:  # sums of some hundred terms in another order, over 6 steps
        assert np.abs(out[0] - o).max() <= 1e-11 * np.abs(out[0]).max()


@pytest.mark.parametrize("precision,big", [("fp32", 3e38), ("fp64", 1e308)])
@pytest.mark.parametrize("comp", [0, 1, 2])
def test_a_non_finite_push_is_reported(hpic, precision, big, comp):
    d = _workload((32, 9, 7), 0.0)
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
