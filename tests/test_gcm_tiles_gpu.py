"""The layer around the memory unit in BF16 where its tiles and token runs can
go wrong: feature counts that are no multiple of 256 (128-wide tiles), token
counts around tile edges and around the 512-token runs of the weight
gradients, biases and gate at addresses that are 4-byte aligned only.  Forward
and reverse mode against the FP64 oracle at the BF16 gate of the other parity
tests."""
import numpy as np
import pytest
import torch

import oracle as orc
from gpu_util import TOL, check, host
from workloads import make_layer_inputs

pytestmark = pytest.mark.gpu


def unaligned(x):
    """float32 vector one element past a 16-byte boundary."""
    t = torch.zeros(x.size + 1, device="cuda")
    t[1:] = torch.from_numpy(x).cuda()
    return t[1:]


@pytest.mark.parametrize("N,H,M", [
    (257, 2, 129),     # one run, one row past a tile
    (1055, 6, 400),    # D = 384: 128-wide tiles, two runs, a ragged last slice
    (1600, 4, 1600),   # D = 256, three runs
    (2945, 16, 1000),  # D = 1024, five runs of 18 or 19 slices
])
def test_layer(gpu, N, H, M):
    from paper_2604_08542_amd import ops
    d, h, eta, D = 64, 128, 0.05, 64 * H
    x = make_layer_inputs(N, H, d, h, seed=N + H, io_dtype="bf16")
    dY = torch.from_numpy(np.random.default_rng(N).standard_normal((N, D)).astype(np.float32)).to(torch.bfloat16)
    g = {k: torch.from_numpy(x[k]).cuda().to(torch.bfloat16) for k in ("X", "Wqkv", "Wo")}
    w = [torch.from_numpy(x[k]).cuda() for k in ("W1", "W2")]
    b = {k: unaligned(x[k]) for k in ("bqkv", "bo")}
    a = (g["X"], g["Wqkv"], g["Wo"], unaligned(x["alpha"]), *w, eta, M)
    f = ops.gcm_fwd(*a, **b)
    r = ops.gcm_bwd(*a, dY.cuda(), **b)
    torch.cuda.synchronize()
    ra = (x["X"], x["Wqkv"], x["Wo"], x["alpha"], x["W1"], x["W2"], eta, M)
    rb = dict(bqkv=x["bqkv"], bo=x["bo"])
    check("Y", host(f["Y"]), orc.gcm_layer_forward(*ra, **rb)["Y"], TOL["bf16"])
    ref = orc.gcm_layer_backward(*ra, dY.float().numpy(), **rb)
    for k in ("dX", "dWqkv", "dbqkv", "dWo", "dbo", "dalpha", "dW1_0", "dW2_0"):
        check(k, host(r[k]), ref[k], TOL["bf16"])
