"""The layer's reverse mode in BF16 where the gate's product takes its larger
tiles (three and four 32-row blocks per wave; test_gcm_tiles_gpu.py: one), with
a row count that is no multiple of 32: the column sums behind dalpha and dbo
follow the tile's rows.  A query of the dispatch pins the choice.  Against the
FP64 oracle at the BF16 gate of the other parity tests."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as orc
from gpu_util import TOL, check, host
from paper_2604_08542_amd import _lib as L
from workloads import make_layer_inputs

CASES = [(2101, 32, 192), (12505, 16, 256)]  # tokens, heads, rows of the tiles


def test_choice():
    for N, H, rows in CASES:
        assert L.load().ttt_internal_gemm_tile(N, 64 * H, 1, ctypes.c_int64(64 * H)) == rows


@pytest.mark.gpu
@pytest.mark.parametrize("N,H", [c[:2] for c in CASES])
def test_layer(gpu, N, H):
    from paper_2604_08542_amd import ops
    d, h, eta, D, M = 64, 128, 0.05, 64 * H, 5000
    x = make_layer_inputs(N, H, d, h, seed=N + H, io_dtype="bf16")
    dY = torch.from_numpy(np.random.default_rng(N).standard_normal((N, D)).astype(np.float32)).to(torch.bfloat16)
    g = {k: torch.from_numpy(x[k]).cuda().to(torch.bfloat16) for k in ("X", "Wqkv", "Wo")}
    w = [torch.from_numpy(x[k]).cuda() for k in ("alpha", "W1", "W2")]
    b = {k: torch.from_numpy(x[k]).cuda() for k in ("bqkv", "bo")}
    r = ops.gcm_bwd(g["X"], g["Wqkv"], g["Wo"], *w, eta, M, dY.cuda(), **b)
    torch.cuda.synchronize()
    ref = orc.gcm_layer_backward(x["X"], x["Wqkv"], x["Wo"], x["alpha"], x["W1"], x["W2"], eta, M, dY.float().numpy(),
                                 bqkv=x["bqkv"], bo=x["bo"])
    for k in ("dX", "dWqkv", "dbqkv", "dWo", "dbo", "dalpha", "dW1_0", "dW2_0"):
        check(k, host(r[k]), ref[k], TOL["bf16"])
