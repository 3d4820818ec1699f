"""The FP32 push's 1/sqrt(s) is the correctly rounded square root followed by the correctly
rounded reciprocal, for every s in [1, 4): every significand with either parity of the
exponent, beyond which both only scale.  Read off a move of 2^-31 / gamma cells from a cell
edge, which is exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

F = np.float32


def _momenta(s):
    """u2, u3 with 1 + u2 u2 + u3 u3 = s after every rounding."""
    k = np.floor(8 * np.sqrt(s.astype(float) - 1))
    return (k / 8).astype(F), np.sqrt(s.astype(float) - 1 - k * k / 64).astype(F)


def _check(hpic, u2, u3):
    n1, n2, n = 8, 4096, u2.size
    with np.errstate(over="ignore"):
        s = (F(1) + u2 * u2) + u3 * u3
        want = F(1) / np.sqrt(s)
    sim = hpic.Sim([hpic.config(n1, n2, 0.25, 1.0, 0.125, precision="fp32")])
    x = np.stack([np.zeros(n), np.arange(n) % n2 + 0.5])
    sim.set_particles(0, x, np.stack([np.full(n, 2.0**-30), u2, u3]), np.full(n, 1e-9))
    sim.step(1)
    p = sim.particles(0)
    sim.close()
    got = np.empty(n)
    got[p["id"]] = p["x"][0]
    bad = np.flatnonzero(got * 2.0**33 != want)
    assert bad.size == 0, (s[bad[:5]], got[bad[:5]] * 2.0**33, want[bad[:5]])


@pytest.mark.parametrize("part", range(4))
def test_every_significand(hpic, part):
    lo = int(F(1).view(np.int32))
    s = (lo + part * 2**22 + np.arange(2**22)).astype(np.int32).view(F)
    u2, u3 = _momenta(s)
    assert np.array_equal((F(1) + u2 * u2) + u3 * u3, s)
    _check(hpic, u2, u3)


def test_up_to_infinity(hpic):
    u3 = np.exp2(np.random.default_rng(5).uniform(0, 64.5, 2**20)).astype(F)
    _check(hpic, np.zeros_like(u3), u3)
