"""The fused block ahead of the state passes that run many sequence-heads side
by side: enough of them, on every shape of the dispatch, against the oracle
prologue composed with the oracle rule (metric and bar of
tests/test_gpu_fused_block.py; the plain forward, which keeps the rule's q, k
and v in its workspace, against the saving one bit for bit).  Ragged lengths of
several chunks, packed input with sequences shorter than the convolution,
every width, with and without an initial state."""
import numpy as np
import pytest
import torch

from tests.test_gpu_fused_block import G, compare, fused_inputs, refs, say  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu

LENS = [64, 0, 1, 2, 79, 128, 330, 130]


@pytest.mark.parametrize("dk,dv,B,H,T,width,h0_std", [
    (64, 64, 8, 13, 144, 4, 0.02),
    (64, 64, 8, 13, 330, 1, None),
    (128, 128, 10, 6, 129, 4, None),
    (128, 128, 10, 6, 330, 3, 0.02),
    (128, 128, 11, 16, 130, 2, 0.02),
    (256, 512, 2, 6, 330, 4, 0.02),
    (256, 512, 3, 14, 100, 3, 0.02),
    (256, 512, 3, 14, 300, 4, None),
])
def test_fused_chain_dense(G, refs, dk, dv, B, H, T, width, h0_std):  # noqa: F811
    inp = fused_inputs(B, T, H, dk, dv, seed=51, width=width, h0_std=h0_std)
    compare(G, refs, inp, "fused_chain_%d_%dx%d" % (dk, B * H, T))


# 16 chunks, 6 of them the longest sequence's: 16 H / 6 chains side by side
@pytest.mark.parametrize("dk,dv,H,width", [(64, 64, 52, 4), (64, 64, 52, 2), (128, 128, 26, 4),
                                           (128, 128, 96, 3), (256, 512, 8, 4), (256, 512, 22, 4)])
def test_fused_chain_packed(G, refs, dk, dv, H, width):  # noqa: F811
    cu = np.concatenate([[0], np.cumsum(LENS)]).astype(np.int32)
    inp = fused_inputs(1, int(cu[-1]), H, dk, dv, seed=52, width=width, cu=cu)
    compare(G, refs, inp, "fused_chain_packed_%d_%d" % (dk, H))


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("dk,dv,B,H", [(64, 64, 8, 13), (128, 128, 10, 6), (256, 512, 2, 6)])
def test_fused_chain_both_backward_forms(G, refs, mode, dk, dv, B, H):  # noqa: F811
    lib = G.load_library()
    inp = fused_inputs(B, 150, H, dk, dv, seed=53)
    prev = lib.gdn_debug_block_bwd(mode)
    try:
        compare(G, refs, inp, "fused_chain_form%d_%d" % (mode, dk))
    finally:
        lib.gdn_debug_block_bwd(prev)


@pytest.mark.parametrize("dk,dv,B,H,T", [(64, 64, 8, 13, 300), (128, 128, 10, 6, 300),
                                         (128, 128, 11, 16, 300), (256, 512, 2, 6, 300),
                                         (256, 512, 8, 6, 1024)])
def test_plain_forward_keeps_any_of_q_k_v(G, dk, dv, B, H, T):  # noqa: F811
    """The plain forward with none, one, two or all of the rule's q, k and v
    asked for: the same o and ht as the saving forward, bit for bit."""
    inp = fused_inputs(B, T, H, dk, dv, seed=54)
    d = {n: x.cuda() for n, x in inp.items()}
    say("plain", dk, dv, B, H, T)
    args = [d[n] for n in ("xq", "xk", "xv", "wq", "wk", "wv", "beta", "log_alpha")]
    want = G.gdn_block_fwd(*args, h0=d["h0"], save=True)
    for asked in ((), ("q",), ("k", "v"), ("q", "k", "v")):
        room = {n: torch.empty_like(want[n]) for n in asked}
        got = G.gdn_block_fwd(*args, h0=d["h0"], **room)
        torch.cuda.synchronize()
        for n in ("o", "ht") + asked:
            assert torch.equal(got[n], want[n]), (asked, n)
