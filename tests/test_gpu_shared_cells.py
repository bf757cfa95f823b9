"""Small meshes, where the four waves of a right-hand-side block share 64 cells: against the
oracle and against the general kernel (DG_SEPARATE_STAGE keeps it).

The two kernels add the same terms in another order, and both have the parity bars of the other
tests: 1e-12 in FP64 and 1e-5 in FP32, in the field norms.  The shapes are the edges of a block
(one cell, one below and above 64 cells, several blocks of which the last is ragged, x lines that
are whole waves) and of the rule (the largest shared meshes, and one cell more, which runs the
general kernel and so gives the same bits).
"""
import numpy as np
import pytest
import torch

import oracle
import synthetic
from gpu_util import dev, field_rel, host, make
from paper_2401_06841_amd import dg

pytestmark = pytest.mark.gpu
BASE = dg.DG_AV | dg.DG_PRIM_PROJ | dg.DG_POS_LIMITER
FORCE = BASE | dg.DG_FORCING | dg.DG_FORCE_MEANFREE
TOL = {dg.DG_FP64: 1e-12, dg.DG_FP32: 1e-5}


def _contexts(shape, k, flags, precision, modes):
    ctxs = [make(*shape, k, flags | more, precision) for more in (0, dg.DG_SEPARATE_STAGE)]
    if flags & dg.DG_FORCING:
        for c in ctxs:
            dg.dg_set_forcing(c, modes)
    return ctxs


def _rhs(ctx, u, dt):
    ud = dev(u, ctx)
    out = torch.full_like(ud, float("nan"))
    dg.dg_rhs(ctx, ud, out, dt)
    return host(out)


@pytest.mark.parametrize("precision", [dg.DG_FP64, dg.DG_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("k", [1, 2, 3])
@pytest.mark.parametrize("shape,flags", [
    ((1, 1, 1), BASE), ((9, 7, 1), FORCE), ((64, 1, 1), FORCE), ((13, 5, 1), FORCE | dg.DG_HLLC),
    ((64, 4, 3), FORCE), ((11, 7, 9), dg.DG_POS_LIMITER), ((11, 7, 9), FORCE & ~dg.DG_PRIM_PROJ),
    ((11, 7, 9), FORCE & ~dg.DG_AV), ((8, 8, 12), BASE | dg.DG_HLLC)])
def test_against_oracle_and_general(shape, flags, k, precision):
    print(f"shared cells {shape} k={k} flags={flags} precision={precision}", flush=True)
    u = synthetic.turbulent_like(*shape, k, mach=3.0, seed=k + sum(shape), high_amp=0.02, kmax_frac=0.125)
    if precision == dg.DG_FP32:
        u = u.astype(np.float32).astype(np.float64)
    modes = synthetic.forcing_table(5, amp=5.0)
    cfg = oracle.Cfg(*shape, k, flags=flags)
    dt = oracle.dt_max(cfg, u)
    ref = oracle.rhs(cfg, u, dt, modes if flags & dg.DG_FORCING else None)
    ctxs = _contexts(shape, k, flags, precision, modes)
    got, gen = (_rhs(c, u, dt) for c in ctxs)
    assert max(field_rel(dt * got, dt * ref, u)) < TOL[precision]
    assert max(field_rel(dt * got, dt * gen, u)) < TOL[precision]
    # a step: the stages read the kernel's partial sums (one set per 64 cells) and its failure flag
    out = []
    for c in ctxs:
        ud = dev(u, c)
        status, nxt = dg.dg_rk_step_next(c, ud, 0.5 * dt, False)
        assert status == dg.DG_OK
        out.append((host(ud), nxt))
    assert max(field_rel(out[0][0], out[1][0], u)) < TOL[precision]
    assert out[0][1] == pytest.approx(out[1][1], rel=10 * TOL[precision])


@pytest.mark.parametrize("shape,precision,shared", [
    ((64, 32, 24), dg.DG_FP64, True), ((199, 19, 13), dg.DG_FP64, False), ((64, 32, 24), dg.DG_FP32, True),
    ((199, 19, 13), dg.DG_FP32, True), ((64, 32, 32), dg.DG_FP32, True), ((65537, 1, 1), dg.DG_FP32, False)])
def test_edges_of_the_rule(shape, precision, shared):
    print(f"rule edge {shape} precision={precision}", flush=True)
    k = 1
    u = synthetic.turbulent_like(*shape, k, mach=3.0, seed=3, high_amp=0.02, kmax_frac=0.125)
    if precision == dg.DG_FP32:
        u = u.astype(np.float32).astype(np.float64)
    ctxs = _contexts(shape, k, FORCE, precision, synthetic.forcing_table(5, amp=5.0))
    dt = dg.dg_dt_max(ctxs[1], dev(u, ctxs[1]))
    states = [dev(u, c) for c in ctxs]
    nexts = [dg.dg_rk_step_next(c, x, 0.5 * dt, False) for c, x in zip(ctxs, states)]
    assert all(status == dg.DG_OK for status, _ in nexts)
    if shared:
        assert max(field_rel(host(states[0]), host(states[1]), u)) < TOL[precision]
        assert nexts[0][1] == pytest.approx(nexts[1][1], rel=10 * TOL[precision])
    else:
        assert torch.equal(states[0], states[1]) and nexts[0][1] == nexts[1][1]
    # the time step of the kept projection is the one of the state
    assert nexts[0][1] == dg.dg_dt_max(ctxs[0], states[0])
    got, gen = (_rhs(c, u, dt) for c in ctxs)
    if shared:
        assert max(field_rel(dt * got, dt * gen, u)) < TOL[precision]
    else:
        assert np.array_equal(got, gen)
