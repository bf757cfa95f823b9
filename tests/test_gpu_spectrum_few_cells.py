"""The velocity spectrum of meshes whose x lines hold few points or few cells: 16 and more samples
per cell, whose points the threads of a block share (15 as the neighbour below), and short lines, of
which a block takes more (with an odd count of lines left over), against the oracle.

The bar is that of the other spectrum tests: 1e-12 of the total energy plus 1e-9 of the shell.
"""
import numpy as np
import pytest

import oracle
import synthetic
from gpu_util import dev, make
from paper_2401_06841_amd import dg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,k,p", [
    ((1, 1, 1), 1, 90), ((1, 2, 1), 3, 75), ((2, 1, 2), 2, 60), ((3, 2, 2), 3, 16), ((3, 2, 2), 2, 15), ((8, 4, 2), 1, 25),
    ((16, 2, 1), 3, 32), ((1, 1, 1), 2, 128), ((4, 48, 48), 2, 4), ((8, 75, 75), 1, 1), ((4, 45, 45), 3, 3)])
@pytest.mark.parametrize("precision", [dg.DG_FP64, dg.DG_FP32], ids=["fp64", "fp32"])
def test_spectrum_of_few_cells_a_line(shape, k, p, precision):
    print(f"spectrum few cells {shape} k={k} p={p} precision={precision}", flush=True)
    u = synthetic.turbulent_like(*shape, k, mach=3.0, seed=sum(shape) + p, high_amp=0.02, kmax_frac=0.125)
    if precision == dg.DG_FP32:
        u = u.astype(np.float32).astype(np.float64)
    ctx = make(*shape, k, 0, precision)
    got = dg.dg_velocity_spectrum(ctx, dev(u, ctx), p)
    ref = oracle.velocity_spectrum(oracle.Cfg(*shape, k), u, p)
    assert got.shape == ref.shape
    assert np.all(np.abs(got - ref) <= 1e-12 * ref.sum() + 1e-9 * np.abs(ref))
