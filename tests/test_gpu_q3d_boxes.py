"""Tiles, boxes and the cell order of the quasi-3D push: every mode count and
tile size against the oracle, and sorted runs against unsorted ones whose boxes
outgrow the LDS or wrap around the grid."""
import numpy as np
import pytest

import oracle
from test_gpu_q3d_particles import _by_id, _particles, _plasma, _random_fields, _read_fields, _zdiff

pytestmark = pytest.mark.gpu


def _make(hpic, prec, M, n1, n2=17, ppc=(2, 2, 2), uth=0.1, drift=0.0, seed=3):
    gen = np.random.default_rng(seed)  # 40 steps of light fall short of the wall
    x, u, w = _plasma(gen, n1, n2, 0.2, 0.25, n2 - 10, ppc=ppc, uth=uth, drift=drift)
    E, B = (_random_fields(gen, M, n1, n2, 0.1) for _ in range(2))
    B[:, 1, 0] = 0
    if M > 1:
        B[1, 1, 0] = 0.1 * gen.standard_normal(n1)
    sim = hpic.Sim([hpic.config(n1, n2, 0.2, 0.25, 0.04, alpha=0.5, precision=prec, modes=M)])
    for m in range(M):
        sim.set_fields_mode(0, m, E[m], B[m])
    sim.set_particles(0, x, u, w, q_over_m=-1.0, q=-1.0)
    st = oracle.StateQ(oracle.gridq(n1, n2, M, 0.2, 0.25, 0.04, alpha=0.5), -1.0, x, u, -w, E, B)
    return sim, st


# bins of sbz columns give tiles of 4 to 16 columns; five modes and more shrink
# them further.  The tolerances are those of the one-step
# test against the oracle: rounding of the form, with sums over more modes.
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-11), ("fp32", 3e-5)])
@pytest.mark.parametrize("M,sbz", [(1, 1), (1, 4), (2, 2), (2, 4), (3, 1), (4, 2), (5, 4), (8, 4), (8, 1)])
def test_modes_and_tiles_match_oracle(hpic, prec, tol, M, sbz):
    sim, st = _make(hpic, prec, M, 32)
    sim.set_tiling(sbz, 2, 1)
    sim.step(2)
    st.step(2)
    x, u = _particles(sim)
    assert np.abs(_zdiff(x[0], st.pos[0], 6.4)).max() <= tol * 10 * 0.2
    assert np.abs(x[1:] - np.stack(st.pos[1:])).max() <= tol * 10 * 17 * 0.25
    scale = np.abs(st.J).max()
    for m in range(M):
        for c in range(3):
            assert np.abs(sim.current_mode(0, c, m) - st.J[m, c]).max() <= tol * 10 * scale
    sim.close()


@pytest.mark.parametrize("n1,M,sbz,ppc,uth,drift",
                         [(16, 3, 4, (2, 2, 2), 0.1, 0.0), (8, 2, 4, (2, 2, 2), 0.3, 1.0),
                          (64, 3, 4, (6, 5, 3), 0.1, 0.0), (64, 1, 2, (2, 2, 2), 0.3, 3.0),
                          (64, 4, 3, (2, 2, 2), 0.5, 0.0), (32, 6, 4, (2, 2, 2), 0.2, 1.0)])
def test_order_and_boxes_leave_the_bits(hpic, n1, M, sbz, ppc, uth, drift):
    """FP32 form (integer deposit): a sort on every step, on every seventh and
    none give the same bits, over 40 steps in which unsorted boxes outgrow the
    LDS and pass the periodic edge; cells of 90 particles pass the order's table."""
    ref = None
    for K in (1024, 1, 7):
        sim, _ = _make(hpic, "fp32", M, n1, ppc=ppc, uth=uth, drift=drift)
        sim.set_tiling(sbz, 2, K)
        sim.step(40)
        p = _by_id(sim.particles(0))
        got = [*_read_fields(sim, M), p["x"], p["u"]]
        sim.close()
        ref = ref or got
        for a, b in zip(got, ref):
            assert np.array_equal(a, b), K


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_a_new_tiling_sorts_before_the_next_step(hpic, prec):
    a, _ = _make(hpic, prec, 3, 64)
    b, _ = _make(hpic, prec, 3, 64)
    for k, sbz in enumerate((4, 1, 2, 4)):
        a.set_tiling(sbz, 2, 16)
        a.step(3)
        b.step(3)
        (Ea, Ba), (Eb, Bb) = _read_fields(a, 3), _read_fields(b, 3)
        if prec == "fp32":
            assert np.array_equal(Ea, Eb) and np.array_equal(Ba, Bb)
        else:  # FP64 atomics: sums of some hundred terms in another order
            assert max(np.abs(Ea - Eb).max(), np.abs(Ba - Bb).max()) <= 1e-11 * np.abs(Eb).max()
    a.close()
    b.close()
