"""The inner loss of a long chunk at large state sizes with BF16 products: 67
million equal squares, whose rounding errors do not cancel.  With W2 = 0 and V
not normalised every residual is -v, so the loss is d v^2.  The sum's longest
runs are the 32 squares of a lane's strip, its 16 strips, 8 wave partials and 8
levels of a tree, so 64 roundings of 2^-24 bound its relative error; in one run
per lane this v loses three times that."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_loss_of_a_long_chunk(gpu):
    from paper_2604_08542_amd import ops
    N, d, h, v = 262144, 256, 128, 1.4153239727020264
    K = torch.ones((N, 1, d), device="cuda")
    W1 = torch.ones((1, d, h), device="cuda") / d
    W2 = torch.zeros((1, h, d), device="cuda")
    r = ops.chunk_fwd(K, K, torch.full_like(K, v), W1, W2, 0.5, N, norm=(True, True, False), emit_loss=True,
                      mma_bf16=True)
    exact = d * float(torch.tensor(v, dtype=torch.float32)) ** 2
    assert abs(float(r["loss"][0, 0]) / exact - 1) <= 64 * 2.0 ** -24
