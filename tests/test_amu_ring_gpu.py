"""Chain reverse mode of the paper's unit around the number of chunks whose
operand copies stay in the workspace (a ring of five sets of weights in BF16,
of two in FP32): as many sets as the ring holds, one more, and twice around.
Against the FP64 oracle at the gates of the other parity tests."""
import numpy as np
import pytest
import torch

import oracle as orc
from gpu_util import TOL, check, host, to_dev
from workloads import make_eta_tok, make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h", [128, 256])
@pytest.mark.parametrize("C,io", [(1, "f32"), (2, "f32"), (5, "f32"), (4, "bf16"), (5, "bf16"), (11, "bf16")])
def test_chain(gpu, C, io, h):
    from paper_2604_08542_amd import ops
    M, H, d = 70, 2, 64
    N = C * M - 7
    x = make_inputs(N, H, d, h, seed=C + h, io_dtype=io, with_dO=True)
    x["W3"] = (np.random.default_rng(C).standard_normal(x["W1"].shape) / np.sqrt(d)).astype(np.float32)
    x["eta"] = make_eta_tok(N, H, M, 20.0, 3)
    Q, K, V, dO = (to_dev(x[k], io) for k in ("Q", "K", "V", "dO"))
    w = [torch.from_numpy(x[k]).cuda() for k in ("eta", "W1", "W2", "W3")]
    g = ops.amu_bwd(Q, K, V, *w, M, dO)
    torch.cuda.synchronize()
    ref = orc.ttt_backward_swiglu(x["Q"], x["K"], x["V"], x["W1"], x["W2"], x["W3"], x["eta"], M, x["dO"])
    for k in ("dQ", "dK", "dV", "dW1_0", "dW2_0", "dW3_0"):
        check(k, host(g[k]), ref[k], TOL[io])
