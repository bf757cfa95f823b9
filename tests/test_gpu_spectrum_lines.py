"""The velocity spectrum's own transform (grids whose sides have at most 512 points and no prime
factor above 5) and the edge of its rule, against the oracle: every radix alone and in chains of
stages, sides with two real lines per complex one left over, sides at the edges of the block sizes
(256, 384, 512 points), and grids that keep the library's transform (a side of 7 or 520 points, or
too few points along x for the rounded-up frequencies to fit the scratch).

The bar is that of the other spectrum tests: 1e-12 of the total energy plus 1e-9 of the shell.
"""
import numpy as np
import pytest

import oracle
import synthetic
from gpu_util import dev, make
from paper_2401_06841_amd import dg

pytestmark = pytest.mark.gpu
FLAGS = dg.DG_AV | dg.DG_PRIM_PROJ | dg.DG_POS_LIMITER


@pytest.mark.parametrize("shape,k,p", [
    ((16, 2, 3), 1, 1), ((16, 4, 5), 1, 1), ((18, 6, 8), 2, 1), ((9, 5, 3), 2, 2), ((8, 3, 2), 3, 4), ((25, 2, 2), 1, 5),
    ((64, 4, 3), 3, 8), ((128, 2, 3), 2, 3), ((2, 128, 9), 1, 3), ((5, 3, 128), 2, 3), ((128, 1, 2), 3, 4),
    ((4, 128, 1), 3, 4), ((4, 1, 128), 3, 4), ((4, 64, 65), 1, 4), ((4, 100, 96), 1, 4), ((162, 2, 1), 2, 3), ((8, 2, 125), 2, 4),
    ((7, 8, 4), 2, 1), ((4, 7, 4), 2, 3), ((130, 1, 1), 2, 4), ((3, 4, 5), 1, 1), ((15, 2, 2), 1, 1)])
@pytest.mark.parametrize("precision", [dg.DG_FP64, dg.DG_FP32], ids=["fp64", "fp32"])
def test_spectrum_of_lines(shape, k, p, precision):
    print(f"spectrum lines {shape} k={k} p={p} precision={precision}", flush=True)
    u = synthetic.turbulent_like(*shape, k, mach=3.0, seed=sum(shape) + p, high_amp=0.02, kmax_frac=0.125)
    if precision == dg.DG_FP32:
        u = u.astype(np.float32).astype(np.float64)
    ctx = make(*shape, k, FLAGS, precision)
    got = dg.dg_velocity_spectrum(ctx, dev(u, ctx), p)
    ref = oracle.velocity_spectrum(oracle.Cfg(*shape, k), u, p)
    assert got.shape == ref.shape
    assert np.all(np.abs(got - ref) <= 1e-12 * ref.sum() + 1e-9 * np.abs(ref))
