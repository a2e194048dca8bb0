"""The paper's unit with BF16 products at d = 64 where its tiles can go wrong:
chunks around the 32-token tile and around one tile per work-group, fewer
tiles than work-groups, head counts whose grid is no multiple of 8, both
hidden sizes, float32 and bfloat16 tokens.  Forward and reverse mode against
the FP64 oracle at the BF16 gate of the other parity tests."""
import numpy as np
import pytest
import torch

import oracle as orc
from gpu_util import TOL, check, host, to_dev
from workloads import make_eta_tok, make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sync", ["chain", "gcs"])
@pytest.mark.parametrize("N,M,H,h,io", [
    (33, 31, 1, 256, "bf16"),
    (64, 33, 3, 128, "f32"),
    (289, 128, 3, 256, "f32"),
    (1057, 1024, 2, 128, "bf16"),
    (1700, 600, 16, 256, "bf16"),
])
def test_paper_unit(gpu, N, M, H, h, io, sync):
    from paper_2604_08542_amd import ops
    d = 64
    x = make_inputs(N, H, d, h, seed=N + M, io_dtype="bf16", with_dO=True)
    x["W3"] = (np.random.default_rng(M + 2).standard_normal(x["W1"].shape) / np.sqrt(d)).astype(np.float32)
    x["eta"] = make_eta_tok(N, H, M, 20.0, 3)
    Q, K, V, dO = (to_dev(x[k], io) for k in ("Q", "K", "V", "dO"))
    w = [torch.from_numpy(x[k]).cuda() for k in ("eta", "W1", "W2", "W3")]
    f = ops.amu_fwd(Q, K, V, *w, M, sync=sync, mma_bf16=True)
    g = ops.amu_bwd(Q, K, V, *w, M, dO, sync=sync, mma_bf16=True)
    torch.cuda.synchronize()
    a = (x["Q"], x["K"], x["V"], x["W1"], x["W2"], x["W3"], x["eta"], M)
    ref = orc.ttt_forward_swiglu(*a, sync=sync)
    refb = orc.ttt_backward_swiglu(*a, x["dO"], sync=sync)
    for k in ("O", "W1_T", "W2_T", "W3_T"):
        check(k, host(f[k]), ref[k], TOL["bf16"])
    for k in ("dQ", "dK", "dV", "dW1_0", "dW2_0", "dW3_0"):
        check(k, host(g[k]), refb[k], TOL["bf16"])
    check("deta_tok", host(g["deta_tok"]).T, refb["deta_tok"].T, TOL["bf16"], row_mult=1.0)
