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


# entry point, its trailing arguments, (H, d, h, N, M, io), bytes that have always been enough
LARGE = [
    ("ttt_workspace_bytes", (1,), (1, 256, 128, 1, 1, L.TTT_F32), 1915392),
    ("ttt_workspace_bytes", (1,), (1, 256, 128, 1, 1, L.TTT_BF16), 1353984),
    ("ttt_workspace_bytes", (1,), (1, 4096, 16384, 1, 42, L.TTT_F32), 3263792640),
    ("ttt_workspace_bytes", (1,), (2, 256, 640, 300, 257, L.TTT_F32), 20017664),
    ("ttt_workspace_bytes", (1,), (1, 1024, 4096, 87936, 10992, L.TTT_BF16), 1569899264),
    ("ttt_workspace_bytes", (3,), (1, 256, 16384, 47549, 13471, L.TTT_BF16), 5567414272),
    ("ttt_amu_workspace_bytes", (), (1, 1024, 4096, 27480, 10992, L.TTT_BF16), 728727808),
    ("ttt_amu_bwd_workspace_bytes", (0,), (1, 1024, 4096, 27480, 10992, L.TTT_BF16), 2365784320),
    ("ttt_amu_bwd_workspace_bytes", (1,), (2, 256, 128, 33, 33, L.TTT_BF16), 2523136),
    ("ttt_gcm_workspace_bytes", (), (1, 1024, 4096, 10992, 5496, L.TTT_BF16), 950493952),
]


@pytest.mark.parametrize("name,extra,shape,enough", LARGE)
def test_large_states_take_no_more(lib, name, extra, shape, enough):
    assert 0 < getattr(lib, name)(ctypes.byref(prob(*shape)), *extra) <= enough


@pytest.mark.parametrize("shape,enough", [
    ((16, 64, 128, 2729, 918, L.TTT_BF16), 164739584),
    ((2, 64, 128, 700, 300, L.TTT_BF16), 71534592),
    ((32, 64, 256, 2050, 500, L.TTT_BF16), 323334656),
    ((36, 64, 256, 1540, 500, L.TTT_BF16), 306945536),
    ((24, 64, 128, 1100, 300, L.TTT_BF16), 139938304),
    ((16, 64, 256, 43968, 10992, L.TTT_BF16), 1516417536),
])
def test_layer_reverse_takes_no_more(lib, shape, enough):
    """Shapes whose weight gradients are cut into runs of tokens."""
    assert 0 < lib.ttt_gcm_bwd_workspace_bytes(ctypes.byref(prob(*shape))) <= enough


def test_paper_unit_large_state_holds_what_bf16_touches(lib):
    """BF16 products at 1024 x 4096: per chunk row the forward keeps K, Q, E (6 d
    bytes), V's factor and five hidden rows (10 h); the FP32 form one hidden row
    and V in FP32 more."""
    rows, d, h = 1280, 1024, 4096

    def per_row(io):
        a, b = (lib.ttt_amu_workspace_bytes(ctypes.byref(prob(1, d, h, n, n, io))) for n in (rows, 2 * rows))
        return (b - a) / rows
    assert per_row(L.TTT_BF16) == 6 * d + 4 + 10 * h
    assert per_row(L.TTT_F32) == 12 * d + 4 * d + 24 * h
