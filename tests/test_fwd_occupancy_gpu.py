"""The forward step at h = 128 with FP32 rows on both sides of the number of
work-groups up to which it has a CU's registers to itself (16 heads of 16 and 17
tiles: 256 and 272 work-groups), FP32 and BF16 products.  Against the FP64
oracle at the gates of the other parity tests."""
import pytest
import torch

import oracle as orc
from gpu_util import TOL, check, host, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mma", [False, True])
@pytest.mark.parametrize("M", [512, 530])
def test_forward(gpu, M, mma):
    from paper_2604_08542_amd import ops
    N, H, h = 2 * M + 5, 16, 128
    x, d = inputs(N, H, h, seed=M, io="bf16" if mma else "f32")
    args = [d[k].float() for k in ("Q", "K", "V", "W1", "W2")]
    r = ops.chunk_fwd(*args, 0.1, M, emit_loss=True, mma_bf16=mma)
    torch.cuda.synchronize()
    ref = orc.ttt_forward(x["Q"], x["K"], x["V"], x["W1"], x["W2"], 0.1, M)
    for k in ("O", "loss", "W1_T", "W2_T"):
        check(k, host(r[k]), ref[k], TOL["bf16" if mma else "f32"])
