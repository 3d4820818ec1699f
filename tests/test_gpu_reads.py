"""Field reads through the host come back whole, at sizes around the pieces (2^18
float and 2^17 double values) that they are read in."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,real", [("fp32", np.float32), ("fp64", np.float64)])
@pytest.mark.parametrize("n1,n2", [(8, 4), (512, 255), (512, 256), (512, 257), (512, 512), (512, 513), (1024, 900)])
def test_fields_come_back(hpic, prec, real, n1, n2):
    gen = np.random.default_rng(n2)
    E, B = gen.standard_normal((2, 3, n2, n1))
    sim = hpic.Sim([hpic.config(n1, n2, 0.2, 0.2, 0.05, precision=prec)])
    sim.set_fields(0, E, B)
    got = sim.fields(0)
    assert np.array_equal(got[0], E.astype(real)) and np.array_equal(got[1], B.astype(real))
    sim.close()


@pytest.mark.parametrize("prec,real", [("fp32", np.complex64), ("fp64", np.complex128)])
@pytest.mark.parametrize("n1,n2", [(16, 8), (512, 255), (512, 256)])
def test_modes_come_back(hpic, prec, real, n1, n2):
    gen = np.random.default_rng(n2)
    E, B = gen.standard_normal((2, 3, n2 + 1, n1)) + 1j * gen.standard_normal((2, 3, n2 + 1, n1))
    sim = hpic.Sim([hpic.config(n1, n2, 0.1, 0.1, 0.02, precision=prec, modes=2)])
    sim.set_fields_mode(0, 1, E, B)
    for c in range(3):
        assert np.array_equal(sim.field_mode(0, c, 1), E[c].astype(real))
        assert np.array_equal(sim.field_mode(0, c + 3, 1), B[c].astype(real))
    sim.close()
