"""GELU and its derivative in the network's gradient, value by value against 64 bits.

One row of zero features through zero weights: the second layer's pre-activations are its biases, the
last layer's gradient is g gelu(b) and the second bias's g w3 gelu'(b), with g = 2 (y - t).  With
w3 = 2^-20, |y| below 1e-3 and t = -2^20 the residual rounds to 2^20, so both come out of the kernel
scaled by powers of two, every bit of them.

The bars are the largest errors over |z| <= 8 of the same expressions with correctly rounded erf and
exp in FP32, 4.5e-7 (z (1 + erf)/2) and 1.4e-7 (its derivative).
"""
import math

import numpy as np
import pytest
import torch
from scipy.special import ndtr

from gpu_util import make
from paper_2401_06841_amd import dg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zmax", [0.01, 0.1, 1.0, 3.0, 8.0])
def test_gelu_and_its_derivative(zmax):
    print(f"gelu |z| <= {zmax}", flush=True)
    ctx = make(4, 4, 4, 2, 0)
    rng = np.random.default_rng(3)
    o_b2, o_w3 = 64 * 20 + 64 + 64 * 64, 64 * 20 + 64 + 64 * 64 + 64
    P = torch.zeros(dg.DG_MLP_NPARAM, device="cuda")
    P[o_w3:o_w3 + 64] = 2.0 ** -20
    x, t = torch.zeros((1, 20), device="cuda"), torch.full((1,), -(2.0 ** 20), device="cuda")
    grad, loss = torch.empty_like(P), torch.empty(1, device="cuda")
    zs, fs, ds = [], [], []
    for _ in range(64):
        z = rng.uniform(-zmax, zmax, 64).astype(np.float32)
        P[o_b2:o_b2 + 64] = torch.as_tensor(z, device="cuda")
        dg.dg_mlp_grad(ctx, P, x, t, grad, loss)
        g = grad.cpu().numpy().astype(np.float64)
        zs.append(z.astype(np.float64))
        fs.append(g[o_w3:o_w3 + 64] / 2.0 ** 21)
        ds.append(g[o_b2:o_b2 + 64] / 2.0)
    z, f, d = (np.concatenate(a) for a in (zs, fs, ds))
    ef = np.abs(f - z * ndtr(z))
    ed = np.abs(d - (ndtr(z) + z * np.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi)))
    print(f"largest errors {ef.max():.2e} {ed.max():.2e}, rms {np.sqrt((ef ** 2).mean()):.2e} {np.sqrt((ed ** 2).mean()):.2e}")
    assert ef.max() < 4.5e-7
    assert ed.max() < 1.4e-7
