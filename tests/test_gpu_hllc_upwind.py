"""HLLC where the gas moves faster than sound: the flux of a face is the upwind cell's, so nothing of
a cell, not even a value that is no number, reaches the cells it moves away from.

A uniform flow along one axis with one broken cell: a NaN in its transverse momentum, or in all its
variables.  The cell upstream of it has the right-hand side of the unbroken state, bit for bit; the
one downstream does not.  (With the velocity projection off, so that the broken cell's traces are its
own weights.)
"""
import numpy as np
import pytest
import torch

from gpu_util import make
from paper_2401_06841_amd import dg

pytestmark = pytest.mark.gpu
N = 8


@pytest.mark.parametrize("stage", [0, dg.DG_SEPARATE_STAGE], ids=["small", "general"])
@pytest.mark.parametrize("precision", [dg.DG_FP64, dg.DG_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("whole", [False, True])
def test_nothing_moves_upstream(whole, axis, k, precision, stage):
    print(f"upwind whole={whole} axis={axis} k={k} precision={precision} stage={stage}", flush=True)
    ctx = make(N, N, N, k, dg.DG_HLLC | stage, precision)
    u = ctx.empty_state()
    u.zero_()
    u[0, 0] = 1.0
    u[1 + axis, 0] = 5.0
    u[1 + (axis + 1) % 3, 0] = 0.25
    good, bad = torch.empty_like(u), torch.empty_like(u)
    dg.dg_rhs(ctx, u, good, 0.0)
    c = 3 + N * (3 + N * 3)
    if whole:
        u[:, :, c] = float("nan")
    else:
        u[1 + (axis + 1) % 3, 0, c] = float("nan")
    dg.dg_rhs(ctx, u, bad, 0.0)
    step = N ** axis
    assert torch.isfinite(good).all()
    assert torch.equal(bad[:, :, c - step], good[:, :, c - step])
    assert torch.isnan(bad[:, 0, c + step]).any()
