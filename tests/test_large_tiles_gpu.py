"""BF16 products at large state sizes where their tiles can go wrong: chunks
one row around the 32-, 128-, 192- and 256-row tile edges, hidden sizes that
are no multiple of 256 (128-wide tiles), several heads through strided views.
Forward and reverse mode of both units against the FP64 oracle, at the BF16
gate of the other parity tests (operands rounded to BF16: 2^-9 per rounding,
a handful of roundings per output, 2e-2 normwise)."""
import numpy as np
import pytest
import torch

import oracle as orc
from gpu_util import TOL, check, host, to_dev
from workloads import make_eta_tok, make_inputs

pytestmark = pytest.mark.gpu

# rows of the first chunk, rows of the last, H, d, h
CASES = [
    (31, 1, 1, 256, 128),
    (129, 33, 2, 256, 384),
    (193, 191, 1, 512, 512),
    (257, 255, 1, 256, 640),
    (385, 128, 1, 768, 256),
]


def strided(x, io):
    """[N][H][d] as a view of a wider tensor (token pitch 2 H d + 8)."""
    N, H, d = x.shape
    big = torch.zeros((N, 2 * H * d + 8), device="cuda", dtype=torch.float32 if io == "f32" else torch.bfloat16)
    v = big[:, : H * d].view(N, H, d)
    v.copy_(to_dev(x, io))
    return v


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("M,last,H,d,h", CASES)
def test_mse_unit(gpu, M, last, H, d, h, io):
    from paper_2604_08542_amd import ops
    N, eta = M + last, 0.5
    x = make_inputs(N, H, d, h, seed=M + d, io_dtype="bf16", with_dO=True)
    Q, K, V, dO = (strided(x[k], io) for k in ("Q", "K", "V", "dO"))
    W1, W2 = (torch.from_numpy(x[k]).cuda() for k in ("W1", "W2"))
    f = ops.chunk_fwd(Q, K, V, W1, W2, eta, M, save_ckpt=True, emit_loss=True, mma_bf16=True)
    g = ops.chunk_bwd(Q, K, V, W1, W2, eta, M, f["ckpt"], dO, mma_bf16=True)
    torch.cuda.synchronize()
    ref = orc.ttt_forward(x["Q"], x["K"], x["V"], x["W1"], x["W2"], eta, M)
    refb = orc.ttt_backward(x["Q"], x["K"], x["V"], x["W1"], x["W2"], eta, M, x["dO"])
    for k in ("O", "loss", "W1_T", "W2_T"):
        check(k, host(f[k]), ref[k], TOL["bf16"])
    for k in ("dQ", "dK", "dV", "dW1_0", "dW2_0", "deta"):
        check(k, host(g[k]), refb[k], TOL["bf16"])


@pytest.mark.parametrize("sync", ["chain", "gcs"])
@pytest.mark.parametrize("M,last,H,d,h", CASES)
def test_paper_unit(gpu, M, last, H, d, h, sync):
    from paper_2604_08542_amd import ops
    N = M + last
    x = make_inputs(N, H, d, h, seed=M + d + 1, io_dtype="bf16", with_dO=True)
    x["W3"] = (np.random.default_rng(M + 2).standard_normal(x["W1"].shape) / np.sqrt(d)).astype(np.float32)
    x["eta"] = make_eta_tok(N, H, M, 100.0, 3)
    Q, K, V, dO = (strided(x[k], "bf16") for k in ("Q", "K", "V", "dO"))
    w = [torch.from_numpy(x[k]).cuda() for k in ("eta", "W1", "W2", "W3")]
    f = ops.amu_fwd(Q, K, V, *w, M, sync=sync)
    g = ops.amu_bwd(Q, K, V, *w, M, dO, sync=sync)
    torch.cuda.synchronize()
    a = (x["Q"], x["K"], x["V"], x["W1"], x["W2"], x["W3"], x["eta"], M)
    ref = orc.ttt_forward_swiglu(*a, sync=sync)
    refb = orc.ttt_backward_swiglu(*a, x["dO"], sync=sync)
    for k in ("O", "W1_T", "W2_T", "W3_T"):
        check(k, host(f[k]), ref[k], TOL["bf16"])
    for k in ("dQ", "dK", "dV", "dW1_0", "dW2_0", "dW3_0"):
        check(k, host(g[k]), refb[k], TOL["bf16"])
    check("deta_tok", host(g["deta_tok"]).T, refb["deta_tok"].T, TOL["bf16"], row_mult=1.0)
