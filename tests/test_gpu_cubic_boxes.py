"""The cubic push's tile boxes: literal column strides (tile widths 8, 16, 32), boxes
that outgrow them or the LDS, the energy-conserving gather, and rejected
particles.  The FP32 form's integer deposit makes every setting bit-identical;
the FP64 form agrees to the rounding of its atomics."""
import numpy as np
import pytest

from paper_1502_01376_amd import workloads as W

pytestmark = pytest.mark.gpu


def _workload(n1, n2, sigma, seed=701):
    return W.drift2d(n1, n2, 0.2, 0.2, 0.1, sub=(2, 2), gamma=8.0, sigma_u=sigma, jitter=True,
                     seed=W.SEED0 + seed, name="cubic boxes")


def _state(sim):
    E, B = sim.fields(0)
    raw = sim.particles_raw(0)
    o = np.argsort(raw["id"])
    return [E, B, sim.current_fixed(0)] + [v[..., o] for _, v in sorted(raw.items())]


@pytest.mark.parametrize("interp", [0, 1])
@pytest.mark.parametrize("n1,n2,sigma", [(64, 32, 0.5), (16, 9, 0.5), (8, 4, 0.1), (128, 21, 4.0)])
def test_every_tile_width_gives_the_same_bits(hpic, n1, n2, sigma, interp):
    d = _workload(n1, n2, sigma)
    ref = None
    # sorted once in 20 steps, a hot plasma outgrows its tiles' literal strides
    for t1, t2, K in [(3, 1, 1), (8, 8, 20), (16, 4, 20), (32, 8, 7), (64, 16, 20), (n1, n2, 20)]:
        sim = hpic.from_workload(d, "fp32", shape=3, interp=interp)
        sim.set_tiling(t1, t2, K)
        sim.step(20)
        got = _state(sim)
        sim.close()
        ref = ref or got
        for a, b in zip(got, ref):
            assert np.array_equal(a, b), (t1, t2, K)


@pytest.mark.parametrize("t1", [8, 16, 32, 64])
def test_fp64_widths_agree(hpic, t1):
    d = _workload(64, 32, 0.5)
    out = []
    for t in (3, t1):
        sim = hpic.from_workload(d, "fp64", shape=3)
        sim.set_tiling(t, 5, 6)
        sim.step(6)
        out.append(np.concatenate(sim.fields(0)))
        sim.close()
    # sums of at most a few hundred terms in another order, over 6 steps
    assert np.abs(out[0] - out[1]).max() <= 1e-11 * np.abs(out[0]).max()


@pytest.mark.parametrize("precision,big", [("fp32", 3e38), ("fp64", 1e308)])
@pytest.mark.parametrize("comp", [0, 1, 2])
def test_a_non_finite_push_is_reported(hpic, precision, big, comp):
    d = _workload(64, 32, 0.0)
    E = np.zeros_like(d["E"])
    E[comp] = big
    sim = hpic.from_workload(d, precision, shape=3)
    sim.set_fields(0, E, d["B"])
    p = sim.particles(0)
    # a charge to mass ratio at which the field's kick overflows
    sim.set_particles(0, p["x"], p["u"], np.abs(p["w"]), q_over_m=-1e4)
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
