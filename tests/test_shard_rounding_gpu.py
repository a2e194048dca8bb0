"""Token shards per chain with FP32 operands where the work-groups that the
device holds do not divide by the chains: rounded down where rounding up would
leave a last round of a few work-groups (48 chains at h = 128), kept rounded up
where the tiles allow no saving (48 chains of 6 tiles), and at h = 256.
Forward and reverse mode against the FP64 oracle at the FP32 gate."""
import numpy as np
import pytest
import torch

import oracle as orc
from gpu_util import TOL, host, inputs, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,H,h,M", [([700, 650, 640], 16, 128, 640), ([352, 385, 360], 16, 128, 192),
                                        ([420, 390, 385], 16, 256, 384)])
def test_uneven_shards(gpu, lens, H, h, M):
    from paper_2604_08542_amd import ops
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    x, d = inputs(cu[-1], H, h, seed=cu[-1] + h, io="f32", with_dO=True)
    f = ops.batched_fwd(d["Q"], d["K"], d["V"], cu, d["W1"], d["W2"], 0.05, M, save_ckpt=True)
    g = ops.batched_bwd(d["Q"], d["K"], d["V"], cu, d["W1"], d["W2"], 0.05, M, f["ckpt"], d["dO"])
    torch.cuda.synchronize()
    for b in range(len(lens)):
        s = slice(cu[b], cu[b + 1])
        ref = orc.ttt_forward(x["Q"][s], x["K"][s], x["V"][s], x["W1"], x["W2"], 0.05, M)
        assert rel(host(f["O"][s]), ref["O"]) <= TOL["f32"], b
    ref = orc.ttt_backward_batched(x["Q"], x["K"], x["V"], cu, x["W1"], x["W2"], 0.05, M, x["dO"])
    for k in ("dQ", "dK", "dV", "dW1_0", "dW2_0"):
        assert rel(host(g[k]), ref[k]) <= TOL["f32"], k
