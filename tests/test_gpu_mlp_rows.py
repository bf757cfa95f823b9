"""The network's gradient at the row counts where its tiles and waves end: one row, one below, at and
above a 16-row tile and the four tiles of a block, one tile per wave of the whole launch (16,384
rows) and one row more, against the FP64 reference.

The bars are those of the bf16 network (3e-2 for the loss, 5e-2 for the norm of each gradient
block).  The targets lie one off the reference outputs, so that the residual, and with it the
gradient, is not a difference of nearly equal numbers at a single row.
"""
import numpy as np
import pytest
import torch

import synthetic
from gpu_util import host, make
from oracle import mlp
from paper_2401_06841_amd import dg
from test_gpu_sensor import ALL, BF16_TOL, _flat, _rows, _unflat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 16383, 16384, 16385])
def test_gradient_at_the_edges_of_tiles(n):
    print(f"gradient rows {n}", flush=True)
    params = synthetic.mlp_params(8)
    P = torch.as_tensor(_flat(params), device="cuda")
    x, _ = _rows(9, min(n, 4000))
    x = np.resize(x, (n, 20)).astype(np.float32)
    y, _ = mlp.forward(params, x.astype(np.float64))
    t = (np.asarray(y).reshape(-1) + np.where(np.arange(n) % 3 == 0, 1.0, -1.0)).astype(np.float32)
    ctx = make(4, 4, 4, 2, ALL)
    grad = torch.full((dg.DG_MLP_NPARAM,), float("nan"), dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    dg.dg_mlp_grad(ctx, P, torch.as_tensor(x, device="cuda"), torch.as_tensor(t, device="cuda"), grad, loss)
    gr = mlp.backward(params, x.astype(np.float64), t.astype(np.float64))
    lr = mlp.loss(params, x.astype(np.float64), t.astype(np.float64))
    assert abs(host(loss)[0] - lr) < BF16_TOL * lr
    for (dW, db), (rW, rb) in zip(_unflat(host(grad)), gr):
        assert np.linalg.norm(dW - rW) / np.linalg.norm(rW) < 5e-2
        assert np.linalg.norm(db - rb) / np.linalg.norm(rb) < 5e-2
