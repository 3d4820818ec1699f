"""What a push costs once the particles have left their tiles: a warm plasma between
two sorts against a cold one that drifts as a whole.  The bounds are several times what
the LDS paths measure, and below what a tile's whole deposit through global memory
costs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _push_us(hpic, cfg, x, u, w, steps):
    sim = hpic.Sim([cfg])
    sim.set_particles(0, x, u, w)
    sim.step(steps)
    sim.profile(True)
    sim.step(2 * steps)
    sim.synchronize()
    ms, n = sim.kernel_times()["push_deposit"]
    sim.close()
    return 1e3 * ms / n


def _cartesian(hpic, prec, sigma, gamma, **kw):
    gen = np.random.default_rng(7)
    n1, n2, ppc, d = 512, 256, 8, 0.2
    x = np.stack([gen.random(n1 * n2 * ppc) * n * d for n in (n1, n2)])
    u = sigma * gen.standard_normal((3, x.shape[1]))
    u[0] += np.sqrt(gamma ** 2 - 1)
    cfg = hpic.config(n1, n2, d, d, 0.08, precision=prec, **kw)
    return _push_us(hpic, cfg, x, u, np.full(x.shape[1], 1e-3 / ppc), 16)


# half of the tiles outgrow the boxes of fields and currents at sigma 0.3, three
# quarters at 1
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [3])
def test_warm_plasma_stays_in_the_lds(hpic, prec, shape):
    cold = _cartesian(hpic, prec, 0.0, 20.0, shape=shape)
    for sigma in (0.3, 1.0):
        warm = _cartesian(hpic, prec, sigma, 1.0, shape=shape)
        assert warm < 4 * cold, (sigma, warm, cold)
