"""BF16 products at large state sizes on every tile that the dispatch can
choose (test_large_tiles_gpu.py: the 128-row ones), with a ragged last row
block.  A query of the dispatch pins the choice, so that other rates cannot
empty a case.  Forward and reverse mode of both units against the FP64 oracle
at the BF16 gate of the other parity tests."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as orc
from gpu_util import TOL, check, host, to_dev
from paper_2604_08542_amd import _lib as L
from workloads import make_eta_tok, make_inputs


def gemm_tile(M, N, nmat, K):
    return L.load().ttt_internal_gemm_tile(M, N, nmat, ctypes.c_int64(K))


def wgrad_tile(*weights):
    col = [(ctypes.c_int32 * len(weights))(*[w[i] for w in weights]) for i in range(3)]
    return L.load().ttt_internal_wgrad_tile(len(weights), *col, 1)


# rows of the first chunk, rows of the last, d, h; rows of the tiles (one
# matrix to the hidden axis, four matrices to it, one to d, two to d), tiles of
# two and of three weight terms
CASES = [
    (801, 33, 256, 16384, (256, 256, 128, 128), 128256, 256256),
    (1057, 7, 256, 16384, (192, 256, 128, 128), 128256, 256256),
    (1601, 70, 4096, 256, (128, 128, 192, 256), 128128, 128128),
    (3201, 5, 4096, 128, (128, 128, 256, 256), 128128, 128128),
]


def test_choice():
    for M, _, d, h, tiles, w2, w3 in CASES:
        assert (gemm_tile(M, h, 1, d), gemm_tile(M, h, 4, d), gemm_tile(M, d, 1, h), gemm_tile(M, d, 2, h)) == tiles
        assert wgrad_tile((d, h, 1), (h, d, 1)) == w2
        assert wgrad_tile((d, h, 1), (d, h, 1), (h, d, 1)) == w3


@pytest.mark.gpu
@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("M,last,d,h", [c[:4] for c in CASES])
def test_mse_unit(gpu, M, last, d, h, io):
    from paper_2604_08542_amd import ops
    N, H, eta = M + last, 1, 0.5
    x = make_inputs(N, H, d, h, seed=M + d, io_dtype="bf16", with_dO=True)
    Q, K, V, dO = (to_dev(x[k], io) for k in ("Q", "K", "V", "dO"))
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


@pytest.mark.gpu
@pytest.mark.parametrize("M,last,d,h", [c[:4] for c in CASES])
def test_paper_unit(gpu, M, last, d, h):
    from paper_2604_08542_amd import ops
    N, H = M + last, 1
    x = make_inputs(N, H, d, h, seed=M + d + 1, io_dtype="bf16", with_dO=True)
    x["W3"] = (np.random.default_rng(M + 2).standard_normal(x["W1"].shape) / np.sqrt(d)).astype(np.float32)
    x["eta"] = make_eta_tok(N, H, M, 100.0, 3)
    Q, K, V, dO = (to_dev(x[k], "bf16") for k in ("Q", "K", "V", "dO"))
    w = [torch.from_numpy(x[k]).cuda() for k in ("eta", "W1", "W2", "W3")]
    f = ops.amu_fwd(Q, K, V, *w, M)
    g = ops.amu_bwd(Q, K, V, *w, M, dO)
    torch.cuda.synchronize()
    a = (x["Q"], x["K"], x["V"], x["W1"], x["W2"], x["W3"], x["eta"], M)
    ref = orc.ttt_forward_swiglu(*a)
    refb = orc.ttt_backward_swiglu(*a, x["dO"])
    for k in ("O", "W1_T", "W2_T", "W3_T"):
        check(k, host(f[k]), ref[k], TOL["bf16"])
    for k in ("dQ", "dK", "dV", "dW1_0", "dW2_0", "dW3_0"):
        check(k, host(g[k]), refb[k], TOL["bf16"])
