"""The state passes that run many sequence-heads side by side, in the ways a
program calls them: sequences long enough that their double buffers wrap and
their loads run two chunks ahead, strong and no decay, beta at its ends, seeded
random problems, HIP graph capture, the no-allocation forward, work on a side
stream.  Against the oracle with the tolerance of the other parity tests, or
bit for bit against the plain calls."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2412_06464_amd.inputs import make_inputs
from tests.test_gpu_graph import REPLAYS, assert_same, block_inputs, capture, refill
from tests.test_gpu_parity import (G, TOL, check_bwd, check_fwd, check_saved, run_bwd, run_fwd,
                                   run_saved, say, to_dev)  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu

# dk, dv, sequences, heads (None: packed LENS): every shape of the dispatch
SHAPES = [(256, 512, 2, 6), (256, 512, 3, 14), (256, 512, None, 6), (256, 512, None, 18),
          (128, 128, 10, 6), (128, 128, 11, 16), (128, 128, None, 24), (128, 128, None, 80),
          (64, 64, 8, 13), (64, 64, None, 48)]
LENS = [300, 0, 64, 1, 500, 130, 448, 79]  # 27 chunks, the longest 8


def problem(dk, dv, B, H, T, seed, **kw):
    if B is None:
        cu = torch.tensor(np.concatenate([[0], np.cumsum(LENS)]), dtype=torch.int32)
        return make_inputs(1, int(cu[-1]), H, dk, dv, "bf16", seed=seed, cu_seqlens=cu, **kw)
    return make_inputs(B, T, H, dk, dv, "bf16", seed=seed, **kw)


@pytest.mark.parametrize("path", ["fwd", "bwd", "saved"])
@pytest.mark.parametrize("dk,dv,B,H", SHAPES)
def test_many_chunks(G, oracle_mod, dk, dv, B, H, path):  # noqa: F811
    """Seven chunks and a ragged tail (dense), one to eight chunks (packed)."""
    inp = problem(dk, dv, B, H, 457, 41, h0_std=0.05, backward=path != "fwd")
    check = dict(fwd=check_fwd, bwd=check_bwd, saved=check_saved)[path]
    check(G, oracle_mod, inp, TOL["bf16"], "many_%s_%d_%s" % (path, dk, B))


@pytest.mark.parametrize("dk,dv,B,H", [(256, 512, 2, 6), (256, 512, 3, 14), (128, 128, 10, 6),
                                       (128, 128, 11, 16), (64, 64, 8, 13)])
@pytest.mark.parametrize("label,kw", [
    ("strong_decay", dict(log_alpha_scale=8.0)),
    ("alpha_one", dict(log_alpha_value=0.0)),
    ("beta_zero", dict(beta_value=0.0, log_alpha_scale=0.05)),
    ("beta_two", dict(beta_value=2.0, log_alpha_scale=0.1)),
])
def test_stress(G, oracle_mod, dk, dv, B, H, label, kw):  # noqa: F811
    inp = problem(dk, dv, B, H, 300, 42, h0_std=0.05, backward=True, **kw)
    check_saved(G, oracle_mod, inp, TOL["bf16"], "stress_%s_%d" % (label, dk))


@pytest.mark.parametrize("seed", range(12))
def test_random(G, oracle_mod, seed):  # noqa: F811
    """Seeded random problems over the lines of the dispatch: dims by turn,
    packed or dense, 12 / 50 / 100 to 5 times as many chains, the gates and the
    initial state there or not; the two backwards agree bit for bit."""
    rng = np.random.default_rng(7000 + seed)
    dk, dv, line = ((64, 64, 100), (128, 128, 50), (256, 512, 12))[seed % 3]
    chains = int(line * rng.uniform(1.0, 5.0))
    kw = dict(h0_std=0.05 if rng.random() < 0.5 else None, backward=True,
              gated=bool(rng.random() < 0.8), log_alpha_scale=float(rng.choice([0.05, 1.0, 4.0])))
    if rng.random() < 0.5:
        lens = [int(rng.integers(0, 400)) for _ in range(int(rng.integers(3, 9)))] + [65]
        chunks = [-(-n // 64) for n in lens]
        H = -(-chains * max(chunks) // sum(chunks)) + 1
        cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
        inp = make_inputs(1, int(cu[-1]), H, dk, dv, "bf16", seed=seed, cu_seqlens=cu, **kw)
    else:
        B, T = int(rng.integers(1, 7)), int(rng.integers(66, 500))
        inp = make_inputs(B, T, -(-chains // B), dk, dv, "bf16", seed=seed, **kw)
    check_saved(G, oracle_mod, inp, TOL["bf16"], "random%d" % seed)
    d = to_dev(inp)
    o, ht = run_fwd(G, d)
    r = run_bwd(G, d)
    o2, ht2, r2 = run_saved(G, d)
    assert torch.equal(o, o2) and torch.equal(ht, ht2)
    for name in r:
        assert torch.equal(r[name], r2[name]), name


@pytest.mark.parametrize("dk,dv,B,H", [(256, 512, 2, 6), (128, 128, None, 24), (64, 64, 8, 13)])
def test_training_step_replays_match_eager(G, dk, dv, B, H):  # noqa: F811
    """Forward, saving forward and saved backward captured as one graph."""
    say("chain_graph", dk, dv, B, H)
    new = lambda seed: to_dev(problem(dk, dv, B, H, 200, seed, h0_std=0.05, backward=True))
    d = new(43)
    host = d["cu_seqlens"].cpu() if d.get("cu_seqlens") is not None else None
    cu = dict(cu_seqlens=d.get("cu_seqlens"), cu_seqlens_host=host)
    args = [d[n] for n in ("q", "k", "v", "beta", "log_alpha")]
    p, keep = G.make_problem(d["q"], d["v"], **cu)
    room = lambda n: torch.empty(n, dtype=torch.uint8, device="cuda")
    ws = [room(f(p)) for f in (G.gdn_chunk_fwd_workspace_size, G.gdn_chunk_fwd_save_workspace_size,
                               G.gdn_chunk_bwd_saved_workspace_size)]
    eager = lambda: _eager_step(G, args, d, cu)
    o, ht, o2, ht2, saved, out = eager()

    def step():
        G.gdn_chunk_fwd(*args, h0=d["h0"], o=o, ht=ht, workspace=ws[0], **cu)
        G.gdn_chunk_fwd_save(*args, h0=d["h0"], o=o2, ht=ht2, saved=saved, workspace=ws[1], **cu)
        G.gdn_chunk_bwd_saved(*args[:4], d["dO"], saved, dht=d["dht"], workspace=ws[2], out=out,
                              **cu)

    step()
    g = capture(step)
    for r in range(REPLAYS):
        refill(d, new(60 + r))
        g.replay()
        torch.cuda.synchronize()
        eo, eht, eo2, eht2, _, ref = eager()
        assert_same(dict(o=o, ht=ht, o2=o2, ht2=ht2), dict(o=eo, ht=eht, o2=eo2, ht2=eht2),
                    "replay %d fwd" % r)
        assert_same({k: out[k] for k in ref}, ref, "replay %d bwd" % r)
    del g, keep


def _eager_step(G, args, d, cu):  # noqa: F811
    o, ht = G.gdn_chunk_fwd(*args, h0=d["h0"], **cu)
    o2, ht2, saved = G.gdn_chunk_fwd_save(*args, h0=d["h0"], **cu)
    out = G.gdn_chunk_bwd_saved(*args[:4], d["dO"], saved, dht=d["dht"], **cu)
    torch.cuda.synchronize()
    return o, ht, o2, ht2, saved, out


@pytest.mark.parametrize("dk,dv,B,H", [(256, 512, 2, 6), (128, 128, 10, 6), (64, 64, 8, 13)])
def test_fused_block_replays_match_eager(G, dk, dv, B, H):  # noqa: F811
    """The fused block's plain and saving forward and its saved backward
    captured as one graph."""
    say("chain_graph_block", dk, dv, B, H)
    d = block_inputs(B, 200, H, dk, dv, 44)
    x = [d[n] for n in ("xq", "xk", "xv", "wq", "wk", "wv")]
    gates = (d["beta"], d["log_alpha"])
    p, _ = G.make_problem(d["xq"], d["xv"], None, None)
    room = lambda n: torch.empty(n, dtype=torch.uint8, device="cuda")
    ws = [room(G.gdn_chunk_fwd_workspace_size(p)), room(G.gdn_chunk_fwd_save_workspace_size(p)),
          room(G.load_library().gdn_block_bwd_saved_workspace_size(ctypes.byref(p), 4))]

    def eager():
        plain = G.gdn_block_fwd(*x, *gates, h0=d["h0"])
        f = G.gdn_block_fwd(*x, *gates, h0=d["h0"], save=True)
        g = G.gdn_block_bwd_saved(*x, f["q"], f["k"], f["v"], d["beta"], d["dO"], f["saved"],
                                  dht=d["dht"])
        torch.cuda.synchronize()
        return plain, f, g

    plain, f, out = eager()

    def step():
        G.gdn_block_fwd(*x, *gates, h0=d["h0"], o=plain["o"], ht=plain["ht"], workspace=ws[0])
        G.gdn_block_fwd(*x, *gates, h0=d["h0"], save=True, o=f["o"], ht=f["ht"], q=f["q"],
                        k=f["k"], v=f["v"], saved=f["saved"], workspace=ws[1])
        G.gdn_block_bwd_saved(*x, f["q"], f["k"], f["v"], d["beta"], d["dO"], f["saved"],
                              dht=d["dht"], workspace=ws[2], out=out)

    step()
    g = capture(step)
    names = ("o", "ht", "q", "k", "v")
    for r in range(REPLAYS):
        refill(d, block_inputs(B, 200, H, dk, dv, 80 + r))
        g.replay()
        torch.cuda.synchronize()
        p2, f2, ref = eager()
        assert_same({k: plain[k] for k in names[:2]}, {k: p2[k] for k in names[:2]}, "plain %d" % r)
        assert_same({k: f[k] for k in names}, {k: f2[k] for k in names}, "saving %d" % r)
        assert_same({k: out[k] for k in ref}, ref, "backward %d" % r)
    del g


@pytest.mark.parametrize("dk,dv,B,H,T", [(256, 512, 2, 6, 457), (128, 128, 10, 6, 457),
                                         (64, 64, 8, 13, 457)])
def test_noalloc_and_side_stream(G, dk, dv, B, H, T):  # noqa: F811
    """The no-allocation forward, and a forward with its backward on a stream
    of its own, give what the plain calls on the current stream give."""
    d = to_dev(problem(dk, dv, B, H, T, 45, h0_std=0.05, backward=True))
    say("chain_noalloc", dk, dv, B, H, T)
    args = [d[n] for n in ("q", "k", "v", "beta", "log_alpha")]
    o, ht, o2, _, _, out = _eager_step(G, args, d, {})
    p, _ = G.make_problem(d["q"], d["v"])
    assert G.gdn_chunk_fwd_workspace_size(p) <= G.NOALLOC_SCRATCH_BYTES
    o3 = torch.full_like(o, float("nan"))
    ht3 = torch.full_like(ht, float("nan"))
    G.gdn_chunk_fwd_noalloc(*args, h0=d["h0"], o=o3, ht=ht3)
    torch.cuda.synchronize()
    assert torch.equal(o3, o) and torch.equal(ht3, ht) and torch.equal(o2, o)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        _, _, o4, ht4, _, out4 = _eager_step(G, args, d, {})
    assert torch.equal(o4, o) and torch.equal(ht4, ht)
    assert_same({k: out4[k] for k in out}, out, "side stream")
