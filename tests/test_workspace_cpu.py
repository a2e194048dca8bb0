"""Sizes of workspaces, pinned so that a call which fitted keeps fitting."""
import ctypes

import pytest

from paper_2604_08542_amd import _lib as L


@pytest.fixture(scope="module")
def lib():
    return L.load()


def prob(H, d, h, N, M, io, flags=7):
    return L.Problem(n_heads=H, d_head=d, d_hidden=h, n_tokens=N, chunk_tokens=M, eta=0.1, flags=flags, io_dtype=io)


@pytest.mark.parametrize("io", [L.TTT_F32, L.TTT_BF16])
@pytest.mark.parametrize("h", [128, 256])
def test_paper_unit_chain_reverse_grows_by_its_weights(lib, h, io):
    """A chunk more costs the FP32 weights before it (three matrices per head)
    and nothing else; the rest is the shard partials, Wh, the weights after the
    last chunk and three sets of six operand copies."""
    H, M = 16, 100
    size = [lib.ttt_amu_bwd_workspace_bytes(ctypes.byref(prob(H, 64, h, C * M, M, io)), L.TTT_SYNC_CHAIN)
            for C in (1, 2, 257)]
    per = H * 3 * 64 * h * 4
    assert size[1] - size[0] == per
    assert size[2] - size[0] == 256 * per
    assert size[0] <= 1024 * 3 * 64 * h * 4 + 3 * per + 3 * H * 6 * 64 * h * 4
