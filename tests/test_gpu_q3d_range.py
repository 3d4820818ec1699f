"""Fields near the largest float: the quasi-3D gather's weights sum to one, so it needs no
range beyond the fields' own."""
import numpy as np
import pytest

from test_gpu_q3d_particles import _by_id, _plasma

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("modes", [1, 3, 6])
@pytest.mark.parametrize("interp", [0, 1])
@pytest.mark.parametrize("prec,big", [("fp32", 2.5e38), ("fp64", 1.2e308)])
def test_a_field_near_the_largest_number_is_gathered(hpic, prec, big, interp, modes):
    """A uniform E_z gives every particle -dt E_z; nothing moves at such a momentum, whose
    square is infinite."""
    n1, n2, dz, dr, dt = 32, 17, 0.2, 0.25, 0.01
    x, u, w = _plasma(np.random.default_rng(3), n1, n2, dz, dr, 7, ppc=(2, 2, 2))
    E = np.zeros((3, n2 + 1, n1), complex)
    E[0] = big
    sim = hpic.Sim([hpic.config(n1, n2, dz, dr, dt, precision=prec, modes=modes, interp=interp)])
    sim.set_particles(0, x, u, w)
    sim.set_fields_mode(0, 0, E, np.zeros_like(E))
    before = _by_id(sim.particles(0))
    sim.step(1)
    after = _by_id(sim.particles(0))
    sim.close()
    assert np.array_equal(before["x"], after["x"])
    # weights along two axes and the kick: a few roundings
    eps = np.finfo(np.float32 if prec == "fp32" else float).eps
    assert np.abs(after["u"][0] / (-dt * big) - 1).max() <= 16 * eps
