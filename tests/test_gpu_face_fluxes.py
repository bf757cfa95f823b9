"""Face fluxes that are one value of the state, bit for bit.

Piecewise constant states that vary along one axis, degree 1, FP32, 16 cells (every weight, factor
and length then is a power of two, so that only the fluxes and their one difference round):
  * HLLC with the flow faster than sound everywhere: the mass flux is the upwind cell's momentum, from
    momentum traces as it stands and from velocity traces with unit density;
  * Rusanov with momentum traces and equal densities: half the sum of the two momenta.
The density's mean weight changes by the difference of two such fluxes over h.
"""
import numpy as np
import pytest
import torch

from gpu_util import make
from paper_2401_06841_amd import dg

pytestmark = pytest.mark.gpu
N = 16


def _rhs(u, flags):
    ctx = make(N, N, N, 1, flags, dg.DG_FP32)
    ud = torch.as_tensor(u, device=ctx.device)
    out = torch.empty_like(ud)
    dg.dg_rhs(ctx, ud, out, 0.0)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _state(axis, rho, m):
    shape = [1, 1, 1]
    shape[2 - axis] = N
    full = lambda a: np.broadcast_to(a.reshape(shape), (N, N, N)).reshape(-1)
    u = np.zeros((4, 4, N ** 3), np.float32)
    u[0, 0], u[1 + axis, 0] = full(rho), full(m)
    return u, full


@pytest.mark.parametrize("stage", [0, dg.DG_SEPARATE_STAGE], ids=["small", "general"])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("prim", [0, dg.DG_PRIM_PROJ], ids=["momenta", "velocities"])
def test_supersonic_hllc_is_the_upwind_momentum(prim, sign, axis, stage):
    print(f"supersonic HLLC prim={prim} sign={sign} axis={axis} stage={stage}", flush=True)
    rng = np.random.default_rng(axis)
    rho = np.ones(N, np.float32) if prim else rng.uniform(0.5, 2.0, N).astype(np.float32)
    m = (sign * rng.uniform(6.0, 9.0, N)).astype(np.float32)
    u, full = _state(axis, rho, m)
    d = np.roll(m, 1) - m if sign > 0 else m - np.roll(m, -1)
    got = _rhs(u, dg.DG_HLLC | prim | stage)
    assert np.array_equal(got[0, 0], full(d * np.float32(N)))


@pytest.mark.parametrize("stage", [0, dg.DG_SEPARATE_STAGE], ids=["small", "general"])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_rusanov_of_equal_densities_is_the_mean_momentum(axis, stage):
    print(f"Rusanov equal densities axis={axis} stage={stage}", flush=True)
    m = np.random.default_rng(axis).uniform(-3.0, 3.0, N).astype(np.float32)
    u, full = _state(axis, np.full(N, 1.3, np.float32), m)
    low, high = np.roll(m, 1) + m, m + np.roll(m, -1)
    got = _rhs(u, stage)
    assert np.array_equal(got[0, 0], full((low - high) * np.float32(N // 2)))
