"""The right-hand side of states whose density is negative at some points of a cell (without the
limiter an expansion may undershoot there): the formula of the viscous pressure goes on, the smaller
of rho nu s and rho (h/p)^2 s / (2 dt), against the oracle.  Caps that bind (a large time step) and
that do not, none (dt = 0), and the learned viscosity; the kernel of small meshes and the general one.

The bars are the right-hand side's: 1e-12 (FP64) and 1e-5 (FP32) in the field norms.
"""
import numpy as np
import pytest
import torch

import oracle
import synthetic
from gpu_util import dev, field_rel, host, make
from paper_2401_06841_amd import dg

pytestmark = pytest.mark.gpu
TOL = {dg.DG_FP64: 1e-12, dg.DG_FP32: 1e-5}
SHAPE = (12, 10, 9)


def _state(k, precision):
    u = synthetic.turbulent_like(*SHAPE, k, mach=3.0, seed=k, high_amp=0.02, kmax_frac=0.2)
    u[0, 1] += 0.9 * u[0, 0]        # the linear mode along x: negative density at low x
    return u.astype(np.float32).astype(np.float64) if precision == dg.DG_FP32 else u


@pytest.mark.parametrize("stage", [0, dg.DG_SEPARATE_STAGE], ids=["small", "general"])
@pytest.mark.parametrize("precision", [dg.DG_FP64, dg.DG_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("dt", [1e-4, 0.05, 0.0])
def test_negative_densities(dt, k, precision, stage):
    print(f"undershoots k={k} dt={dt} precision={precision} stage={stage}", flush=True)
    u = _state(k, precision)
    ref = oracle.rhs(oracle.Cfg(*SHAPE, k, flags=dg.DG_AV), u, dt)
    ctx = make(*SHAPE, k, dg.DG_AV | stage, precision)
    ud = dev(u, ctx)
    out = torch.empty_like(ud)
    dg.dg_rhs(ctx, ud, out, dt)
    assert max(field_rel(host(out), ref, ref)) < TOL[precision]


@pytest.mark.parametrize("stage", [0, dg.DG_SEPARATE_STAGE], ids=["small", "general"])
@pytest.mark.parametrize("precision", [dg.DG_FP64, dg.DG_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("dt", [1e-4, 0.05])
def test_negative_densities_learned_viscosity(dt, precision, stage):
    k = 2
    u = _state(k, precision)
    nc = u.shape[2]
    nu = np.random.default_rng(1).uniform(0.0, 0.1, nc).astype(np.float32).astype(np.float64)
    fb = (np.arange(nc) % 3 == 0).astype(np.int32)
    flags = dg.DG_AV | dg.DG_LEARNED_SENSOR
    ref = oracle.rhs(oracle.Cfg(*SHAPE, k, flags=flags), u, dt, nu=nu, fallback=fb)
    ctx = make(*SHAPE, k, flags | stage, precision)
    ud = dev(u, ctx)
    dg.dg_sensor_set_nu(ctx, torch.as_tensor(nu, device=ctx.device).to(ctx.dtype), torch.as_tensor(fb, device=ctx.device))
    out = torch.empty_like(ud)
    dg.dg_rhs(ctx, ud, out, dt)
    assert max(field_rel(host(out), ref, ref)) < TOL[precision]
