"""The state passes that run many sequence-heads side by side (one chain per
wave), on every shape of their dispatch: enough short sequences that the rule
takes them, against the oracle, with the tolerance of the other parity tests.
Lengths end inside a 16-row tile, on its edge and on a chunk's; packed input
has empty, one-token and one-chunk sequences."""
import numpy as np
import pytest
import torch

from paper_2412_06464_amd.inputs import make_inputs
from tests.test_gpu_parity import (G, TOL, check_bwd, check_fwd, check_saved, run_bwd, run_fwd,
                                   run_saved, to_dev)  # noqa: F401

pytestmark = pytest.mark.gpu

# dk, dv, sequences, heads, tokens (None: packed); sequence-heads side by side
SHAPES = [
    (256, 512, 2, 6, 81, "12: four waves of 16 columns"),
    (256, 512, 3, 14, 65, "42: four waves of 32 columns"),
    (256, 512, None, 14, None, "packed, 32 columns"),
    (128, 128, 10, 6, 129, "60: two workgroups per unit"),
    (128, 128, 11, 16, 63, "176: one workgroup per unit"),
    (128, 128, None, 64, None, "packed, one workgroup per unit"),
    (64, 64, 8, 13, 144, "104"),
    (64, 64, None, 48, None, "packed"),
]


def problem(dk, dv, B, H, T, **kw):
    if B is None:
        lens = [64, 0, 1, 79, 128, 16, 130]
        cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
        return make_inputs(1, int(cu[-1]), H, dk, dv, "bf16", cu_seqlens=cu, **kw)
    return make_inputs(B, T, H, dk, dv, "bf16", **kw)


@pytest.mark.parametrize("dk,dv,B,H,T,what", SHAPES)
@pytest.mark.parametrize("path", ["fwd", "bwd", "saved"])
def test_chain_passes(G, oracle_mod, path, dk, dv, B, H, T, what):
    inp = problem(dk, dv, B, H, T, seed=31, h0_std=0.05, backward=path != "fwd")
    check = dict(fwd=check_fwd, bwd=check_bwd, saved=check_saved)[path]
    check(G, oracle_mod, inp, TOL["bf16"], "chain_%s_%d_%s" % (path, dk, what.split(":")[0]))


@pytest.mark.parametrize("dk,dv,B,H,T", [(256, 512, 3, 14, 100), (128, 128, 10, 6, 100),
                                         (64, 64, 8, 13, 100)])
@pytest.mark.parametrize("kw", [dict(gated=False), dict(log_alpha_scale=0.05, beta_scale=2.0)])
def test_chain_passes_gates(G, oracle_mod, dk, dv, B, H, T, kw):
    """No gates, and weak decay with beta in (0, 2); the saved and the
    stateless backward agree bit for bit, also where the state is absent."""
    inp = problem(dk, dv, B, H, T, seed=32, h0_std=None, backward=True, **kw)
    check_saved(G, oracle_mod, inp, TOL["bf16"], "chain_gates_%d" % dk)
    d = to_dev(inp)
    o, ht = run_fwd(G, d)
    r = run_bwd(G, d)
    o2, ht2, r2 = run_saved(G, d)
    assert torch.equal(o, o2) and torch.equal(ht, ht2)
    for name in r:
        assert torch.equal(r[name], r2[name]), name
