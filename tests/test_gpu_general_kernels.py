"""Kernel families of the step on the meshes and paths that the default rule of a mesh size leaves out.

Meshes of a few ten thousand cells take the kernels whose blocks share 64 cells unless a stage flag is
given, so the general right-hand side and stage kernels are held to the oracle here with
DG_SEPARATE_STAGE: x lines of whole waves (where face moments pass between the lanes of a block), a
failure that shows in the last stage only, the schemes by order (with the five-stage scheme's side
combination) and the learned viscosity.  Then
  * the shared-cells stage kernel against the general one, bit for bit: a driving table off the shell
    keeps the general right-hand side on a small mesh, so nothing else differs;
  * the edges of the shared kernels' rules at FP64 degree 3, where between 32,768 and 49,152 cells a
    shared right-hand side is followed by the general stage kernel;
  * a mean-free FP64 degree-3 step of more than 1,024 right-hand-side blocks, whose mean acceleration
    is reduced by a kernel of its own.
The bars are those of the other tests: 1e-12 in FP64 and 1e-5 in FP32.
"""
import numpy as np
import pytest
import torch

import oracle
import synthetic
from gpu_util import assert_state_close, dev, field_rel, host, make
from paper_2401_06841_amd import dg
from test_gpu_parity import ALL, FORCE, LAST_STAGE_FAILURES, LINE_MESHES, TOL, _oracle_stage_minima

pytestmark = pytest.mark.gpu
FP64, FP32 = dg.DG_FP64, dg.DG_FP32
SEP = dg.DG_SEPARATE_STAGE


def _state(shape, k, precision, seed, mach=3.0, **kw):
    u = synthetic.turbulent_like(*shape, k, mach=mach, seed=seed, **kw)
    return u.astype(np.float32).astype(np.float64) if precision == FP32 else u


@pytest.mark.parametrize("flags", [FORCE, FORCE | dg.DG_HLLC], ids=["rusanov", "hllc"])
@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("mesh,precision", LINE_MESHES + [((11, 9, 7), FP64), ((64, 4, 6), FP32)])
def test_general_rhs(mesh, precision, k, flags):
    print(f"general rhs {mesh} k={k} precision={precision} flags={flags}", flush=True)
    u = _state(mesh, k, precision, k + mesh[1])
    modes = synthetic.forcing_table(5, amp=5.0)
    cfg = oracle.Cfg(*mesh, k, flags=flags)
    dt = oracle.dt_max(cfg, u)
    ctx = make(*mesh, k, flags | SEP, precision)
    dg.dg_set_forcing(ctx, modes)
    ud = dev(u, ctx)
    out = torch.full_like(ud, float("nan"))
    dg.dg_rhs(ctx, ud, out, dt)
    assert max(field_rel(dt * host(out), dt * oracle.rhs(cfg, u, dt, modes), u)) < TOL[precision]


@pytest.mark.parametrize("rel", [0.1, 0.0])
@pytest.mark.parametrize("precision", [FP64, FP32])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_general_last_stage_failure_leaves_state(k, precision, rel):
    print(f"general last-stage failure k={k} precision={precision} rel={rel}", flush=True)
    u = _state((6, 5, 4), k, precision, 0, mach=4.0)
    cfg = oracle.Cfg(6, 5, 4, k, flags=ALL, rho_floor_rel=rel)
    dt = LAST_STAGE_FAILURES[rel][k] * oracle.dt_max(cfg, u)
    m = _oracle_stage_minima(cfg, u, dt)
    assert m[0] > 1e-2 and m[1] > 1e-2 and m[2] < -1e-2, m
    ctx = make(6, 5, 4, k, ALL | SEP, precision, rho_floor_rel=rel)
    ud = dev(u, ctx)
    before = ud.clone()
    assert dg.dg_rk_step(ctx, ud, dt) == dg.DG_RETRY
    assert torch.equal(ud, before)
    rc, dt_next = dg.dg_rk_step_next(ctx, ud, dt, False)
    assert rc == dg.DG_RETRY and dt_next is None
    assert torch.equal(ud, before)
    rc, _ = dg.dg_rk_step_next(ctx, ud, 0.25 * dt, False)
    ref, st = oracle.rk_step(cfg, u, 0.25 * dt)
    assert rc == dg.DG_OK and st == oracle.OK
    assert_state_close(host(ud), ref, TOL[precision], "retried step")


@pytest.mark.parametrize("precision", [FP64, FP32])
@pytest.mark.parametrize("k", [1, 2, 3])
def test_general_schemes_by_order(k, precision):
    shape, flags = (9, 7, 5), FORCE | dg.DG_RK_BY_ORDER
    print(f"general scheme by order k={k} precision={precision}", flush=True)
    u = _state(shape, k, precision, 60 + k, high_amp=0.02, kmax_frac=0.125)
    modes = synthetic.forcing_table(60 + k, amp=2.5)
    cfg = oracle.Cfg(*shape, k, flags=flags)
    ctx = make(*shape, k, flags | SEP, precision)
    dg.dg_set_forcing(ctx, modes)
    ud, dt = dev(u, ctx), oracle.dt_max(cfg, u)
    for i in range(3):
        rc, nxt = dg.dg_rk_step_next(ctx, ud, dt, i > 0)
        u, st = oracle.rk_step(cfg, u, dt, modes)
        assert rc == dg.DG_OK and st == oracle.OK
        dt = oracle.dt_max(cfg, u)
        assert abs(nxt - dt) <= 10 * TOL[precision] * dt
    assert_state_close(host(ud), u, TOL[precision], "scheme by order")


@pytest.mark.parametrize("precision", [FP64, FP32])
def test_general_rhs_with_learned_viscosity(precision):
    n = 10
    u = _state((n, n, n), 2, precision, 13)
    nu, fb = synthetic.random_nu(n ** 3, 1), synthetic.random_fallback(n ** 3, 2)
    if precision == FP32:
        nu = nu.astype(np.float32).astype(np.float64)
    cfg = oracle.Cfg(n, n, n, 2, flags=ALL | oracle.LEARNED)
    dt = oracle.dt_max(cfg, u)
    ctx = make(n, n, n, 2, ALL | dg.DG_LEARNED_SENSOR | SEP, precision)
    ud = dev(u, ctx)
    dg.dg_sensor_set_nu(ctx, torch.as_tensor(nu, device="cuda").to(ctx.dtype), torch.as_tensor(fb, device="cuda"))
    out = torch.empty_like(ud)
    dg.dg_rhs(ctx, ud, out, dt)
    assert max(field_rel(dt * host(out), dt * oracle.rhs(cfg, u, dt, None, nu, fb), u)) < TOL[precision]


# one ragged block, several, whole waves; a rough state on which the limiter acts; both schemes; the
# learned viscosity (degree 2)
STAGES = [(shape, rough, more, k) for k in (1, 2, 3) for shape, rough, more in [
    ((5, 4, 3), False, 0), ((20, 15, 13), False, 0), ((64, 4, 3), False, 0), ((12, 12, 12), True, 0),
    ((12, 12, 12), False, dg.DG_RK_BY_ORDER)]] + [((11, 9, 7), False, dg.DG_LEARNED_SENSOR, 2)]


@pytest.mark.parametrize("precision", [FP64, FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("shape,rough,more,k", STAGES)
def test_shared_stage_kernel_has_the_general_ones_bits(shape, rough, more, k, precision):
    print(f"shared stage bits {shape} k={k} precision={precision} rough={rough} more={more}", flush=True)
    u = _state(shape, k, precision, 9, mach=4.0 if rough else 3.0, high_amp=0.35 if rough else 0.02)
    modes = synthetic.forcing_table_general(5, amp=2.5)
    ctxs = [make(*shape, k, FORCE | more | stage, precision) for stage in (0, SEP)]
    us = [dev(u, c) for c in ctxs]
    nu, fb = synthetic.random_nu(u.shape[2], 1), synthetic.random_fallback(u.shape[2], 2)
    for c in ctxs:
        dg.dg_set_forcing(c, modes)
        if more == dg.DG_LEARNED_SENSOR:
            dg.dg_sensor_set_params(c, torch.zeros(dg.DG_MLP_NPARAM, device="cuda"))
            dg.dg_sensor_set_nu(c, torch.as_tensor(nu, device="cuda").to(c.dtype), torch.as_tensor(fb, device="cuda"))
    dt = (0.25 if rough else 0.5) * dg.dg_dt_max(ctxs[0], us[0])
    for i in range(3):
        (ra, da), (rb, db) = (dg.dg_rk_step_next(c, x, dt, i > 0) for c, x in zip(ctxs, us))
        assert ra == rb == dg.DG_OK
        assert torch.equal(us[0], us[1]), (us[0] - us[1]).abs().max().item()
        assert da == db
        dt = 0.5 * da


# 32,768 cells: shared right-hand side and stage; 33,631: shared right-hand side, general stage kernel;
# 49,152: the largest such mesh; 49,250: both general
@pytest.mark.parametrize("shape,shared", [((32, 32, 32), True), ((199, 13, 13), True), ((64, 32, 24), True),
                                          ((197, 25, 10), False)])
def test_edges_of_the_rules_fp64_k3(shape, shared):
    print(f"rule edges FP64 k=3 {shape}", flush=True)
    k = 3
    u = _state(shape, k, FP64, 3, high_amp=0.02, kmax_frac=0.125)
    modes = synthetic.forcing_table(5, amp=2.5)
    ctxs = [make(*shape, k, FORCE | stage, FP64) for stage in (0, SEP)]
    for c in ctxs:
        dg.dg_set_forcing(c, modes)
    us = [dev(u, c) for c in ctxs]
    dt = 0.5 * dg.dg_dt_max(ctxs[0], us[0])
    outs = [torch.empty_like(x) for x in us]
    for c, x, o in zip(ctxs, us, outs):
        dg.dg_rhs(c, x, o, dt)
    # the two right-hand sides add the same terms in another order
    assert torch.equal(*outs) != shared
    assert max(field_rel(dt * host(outs[0]), dt * host(outs[1]), u)) < TOL[FP64]
    for i in range(2):
        (ra, da), (rb, db) = (dg.dg_rk_step_next(c, x, dt, i > 0) for c, x in zip(ctxs, us))
        assert ra == rb == dg.DG_OK
        assert max(field_rel(host(us[0]), host(us[1]), u)) < TOL[FP64]
        assert da == pytest.approx(db, rel=10 * TOL[FP64]) and da == dg.dg_dt_max(ctxs[0], us[0])
        if not shared:
            assert torch.equal(*us) and da == db


# the rule of the right-hand side at the other degrees and in FP32, by its bits
@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("shape,precision,shared", [
    ((64, 32, 24), FP64, True), ((49153, 1, 1), FP64, False), ((64, 32, 32), FP32, True), ((65537, 1, 1), FP32, False)])
def test_which_right_hand_side_runs(shape, precision, shared, k):
    print(f"right-hand side of {shape} k={k} precision={precision}", flush=True)
    u = _state(shape, k, precision, 3, high_amp=0.02, kmax_frac=0.125)
    outs = []
    for stage in (0, SEP):
        ctx = make(*shape, k, ALL | stage, precision)
        ud = dev(u, ctx)
        outs.append(torch.empty_like(ud))
        dg.dg_rhs(ctx, ud, outs[-1], 1e-5)
    assert torch.equal(*outs) != shared


@pytest.mark.timeout(900)
def test_meanfree_step_above_the_in_stage_reduction_fp64_k3():
    shape, k = (64, 64, 65), 3                    # 1,040 blocks of 256 cells
    print(f"mean-free step {shape} k={k} FP64", flush=True)
    u = _state(shape, k, FP64, 52, high_amp=0.02, kmax_frac=0.125)
    modes = synthetic.forcing_table(15, amp=2.5)
    cfg = oracle.Cfg(*shape, k, flags=FORCE)
    ctx = make(*shape, k, FORCE, FP64)
    dg.dg_set_forcing(ctx, modes)
    ud, dt = dev(u, ctx), oracle.dt_max(cfg, u)
    rc, nxt = dg.dg_rk_step_next(ctx, ud, dt, False)
    assert rc == dg.DG_OK
    ref, st = oracle.rk_step(cfg, u, dt, modes)
    assert st == oracle.OK
    assert_state_close(host(ud), ref, TOL[FP64], "mean-free step")
    d1 = oracle.dt_max(cfg, ref)
    assert abs(nxt - d1) <= 1e-12 * d1
