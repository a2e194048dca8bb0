"""The BF16 reverse step of the MSE unit where its tiles and shards can go
wrong: tokens around the 32-token tile, shards without a tile, an odd number of
shards (at h = 128 two share a work-group when there are more than 256: the last
two cases, 304 shards, 19 per head), both hidden sizes, float32 and bfloat16
tokens.  Against the FP64 oracle at the BF16 gate of the other parity
tests.  d(eta) is left to those: over a few dozen tokens its terms cancel, and
BF16 products alone then move it by more than the gate."""
import pytest
import torch

import oracle as orc
from gpu_util import TOL, host, inputs, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,H,h,io", [
    (33, 31, 1, 256, "bf16"),
    (65, 33, 3, 128, "f32"),
    (289, 128, 3, 256, "f32"),
    (289, 96, 2, 128, "bf16"),
    (700, 225, 2, 128, "f32"),
    (1700, 600, 16, 256, "bf16"),
    (1300, 600, 16, 128, "f32"),
    (1300, 600, 16, 128, "bf16"),
])
def test_reverse_step(gpu, N, M, H, h, io):
    from paper_2604_08542_amd import ops
    x, d = inputs(N, H, h, seed=N + M + H, io=io, with_dO=True)
    f = ops.chunk_fwd(d["Q"], d["K"], d["V"], d["W1"], d["W2"], 0.05, M, save_ckpt=True, mma_bf16=True)
    g = ops.chunk_bwd(d["Q"], d["K"], d["V"], d["W1"], d["W2"], 0.05, M, f["ckpt"], d["dO"], mma_bf16=True)
    torch.cuda.synchronize()
    ref = orc.ttt_backward(x["Q"], x["K"], x["V"], x["W1"], x["W2"], 0.05, M, x["dO"])
    for k in ("dQ", "dK", "dV", "dW1_0", "dW2_0"):
        assert rel(host(g[k]), ref[k]) <= TOL["bf16"], k
