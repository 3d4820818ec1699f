"""The tile sort's division of row numbers and ranks by a tile's sizes, compiled for
the host: exact for every dividend that a grid can give (2^27 rows of 8 cells), from
a float reciprocal that is one unit off either way."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1502_01376_amd", "csrc")
SOURCE = """
#include "hpic_divide.h"
extern "C" void divide(int n, const int *a, int b, float rcp, int *q, int *rem) {
  for (int i = 0; i < n; ++i) q[i] = hp::settle_quotient(a[i], b, (int)((float)a[i] * rcp), rem[i]);
}
"""


@pytest.fixture(scope="module")
def divide(tmp_path_factory):
    d = tmp_path_factory.mktemp("divide")
    src, lib = d / "divide.cpp", d / "divide.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)],
                   check=True)
    fn = ctypes.CDLL(str(lib)).divide

    def run(a, b, rcp):
        q, rem = np.empty_like(a), np.empty_like(a)
        p = [v.ctypes.data_as(ctypes.c_void_p) for v in (a, q, rem)]
        fn(a.size, p[0], b, ctypes.c_float(rcp), p[1], p[2])
        return q, rem
    return run


@pytest.mark.parametrize("b", [1, 2, 3, 5, 7, 8, 10, 300, 1023, 4096])
def test_quotient_and_remainder_are_exact(divide, b):
    gen = np.random.default_rng(b)
    edges = [e + np.arange(-70, 70) for e in (2 ** 22, 2 ** 23, 2 ** 24, 18874367, 2 ** 25, 33554438, 2 ** 26, 2 ** 27)]
    a = np.concatenate([np.arange(4096), *edges, gen.integers(0, 2 ** 27, 200000)]).astype(np.int32)
    rcp = np.float32(1) / np.float32(b)
    for r in (rcp, np.nextafter(rcp, np.float32(0)), np.nextafter(rcp, np.float32(2))):
        q, rem = divide(a, b, r)
        assert np.array_equal(q, a // b) and np.array_equal(rem, a % b)


@pytest.mark.gpu
def test_rows_beyond_the_floats_keep_their_particles(hpic):
    """24 000 001 rows of 8 cells: loading and a new tiling sort the particles of the
    last rows and of random ones, and lose or move none."""
    import torch
    n2 = 24000001
    gen = np.random.default_rng(5)
    rows = np.concatenate([np.arange(n2 - 4000, n2), gen.integers(0, n2, 60000)])
    x = np.stack([gen.random(rows.size) * 8, rows + 0.5])
    sim = hpic.Sim([hpic.config(8, n2, 1.0, 1.0, 0.25)])
    x, u, w = (torch.tensor(v, device="cuda") for v in (x, np.zeros((3, rows.size)), np.ones(rows.size)))
    sim.set_particles_device(0, x, u, w)
    for tile in ((8, 3), (3, 7)):
        sim.set_tiling(*tile, 16)
        p = sim.particles_raw(0)
        o = np.argsort(p["id"])
        assert np.array_equal(p["id"][o], np.arange(rows.size))
        assert np.array_equal(p["cell"][1][o], rows)
        assert np.array_equal(p["cell"][0][o], np.floor(x[0].cpu().numpy()).astype(np.int32))
    sim.close()
