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
                                   run_saved, say, to_dev)  # noqa: F401

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


def training_step(G, d):
    o, ht, r = run_saved(G, d)
    return dict(r, o=o, ht=ht)


PLANTS = [("v", float("nan")), ("v", float("inf")), ("dO", float("nan")), ("dO", float("-inf")),
          ("h0", float("inf")), ("dht", float("nan")), ("dht", float("inf")), ("q", float("nan")),
          ("k", float("inf")), ("beta", float("nan")), ("log_alpha", float("nan"))]


@pytest.mark.parametrize("dk,dv,B,H,T", [(256, 512, 2, 6, 150), (256, 512, 3, 14, 150),
                                         (128, 128, 10, 6, 150), (128, 128, 11, 16, 150),
                                         (64, 64, 8, 13, 150)])
def test_nonfinite_values_reach_no_further(G, dk, dv, B, H, T):
    """A NaN or infinity in one input of one unit changes, of that unit's
    outputs, nothing that it leaves unchanged where the unit is computed alone
    (by the passes that run few sequence-heads), and nothing of any other
    unit: a value of v or dO, above all, stays in its own column of o, ht, dv
    and dh0.  It lies in the middle one of three chunks."""
    inp = problem(dk, dv, B, H, T, seed=33, h0_std=0.05, backward=True)
    b, h = B - 1, H - 2
    cut = lambda x, n: x[b:b + 1, h:h + 1] if n in ("h0", "dht", "dh0", "ht") else x[b:b + 1, :, h:h + 1]
    alone = {n: cut(x, n).contiguous() if isinstance(x, torch.Tensor) else x
             for n, x in inp.items()}
    clean, clean1 = training_step(G, to_dev(inp)), training_step(G, to_dev(alone))
    for name, value in PLANTS:
        say("plant", dk, dv, B * H, name, value)
        planted = {}
        for key, src in (("all", inp), ("one", alone)):
            bb, hh = (b, h) if key == "all" else (0, 0)
            x = src[name].clone()
            at = {2: (bb, hh, dk // 3, dv - 5), 0: (bb, 75, hh)}[2 if name in ("h0", "dht") else 0]
            if x.dim() == 4 and len(at) == 3:
                at = at + (x.shape[3] - 5,)
            x[at] = value
            planted[key] = training_step(G, to_dev(dict(src, **{name: x})))
        for n in clean:
            kept = planted["one"][n] == clean1[n]
            same = planted["all"][n] == clean[n]
            unit = cut(same, n).reshape(kept.shape)
            lost = int((kept & ~unit).sum())
            assert lost == 0, (name, value, n, lost, int(kept.sum()))
            if name in ("v", "dO") and n in ("o", "ht", "dv", "dh0"):
                other = torch.arange(dv, device=unit.device) != dv - 5
                assert bool(unit[..., other].all()), (name, value, n)
            cut(same, n).fill_(True)
            assert bool(same.all()), (name, value, n, "another unit changed")


@pytest.mark.parametrize("dk,dv,H", [(64, 64, 104), (128, 128, 60), (128, 128, 176),
                                     (256, 512, 12)])
@pytest.mark.parametrize("over", ["q", "k", "v", "all", "v_shifted", "ht_v"])
def test_outputs_over_inputs(G, dk, dv, H, over):
    """A forward whose outputs share memory with its inputs gives what it gives
    with buffers of its own: o in the place of q, k, v or one tensor that is
    all three, o on v's rows moved by 64 tokens, ht on v.  The passes read q, k
    and v while they write o and ht, other sequence-heads' and later chunks'
    among them."""
    if over in ("q", "k", "all") and dk != dv:
        pytest.skip("o has v's rows, not q's")
    T = 300
    d = to_dev(problem(dk, dv, 1, H, T, seed=34, h0_std=0.05))
    say("over", dk, dv, H, over)
    if over == "all":
        d["k"] = d["q"] = d["v"] = d["k"]
    elif over == "v_shifted":
        room = torch.empty((1, T + 64, H, dv), dtype=d["v"].dtype, device="cuda")
        d["v"] = room[:, :T].copy_(d["v"])
    elif over == "ht_v":  # v's bytes inside a buffer that holds ht
        n = max(d["v"].numel() * 2, H * dk * dv * 4)
        room = torch.empty(n, dtype=torch.uint8, device="cuda")
        d["v"] = room[:d["v"].numel() * 2].view(d["v"].dtype).view_as(d["v"]).copy_(d["v"])
    want_o, want_ht = run_fwd(G, d)
    keep = {n: d[n].clone() for n in ("q", "k", "v")}
    for save in (False, True):
        for n, x in keep.items():
            d[n].copy_(x)
        kw = dict(h0=d["h0"])
        if over == "v_shifted":
            kw["o"] = room[:, 64:]
        elif over == "ht_v":
            kw["ht"] = room[:H * dk * dv * 4].view(torch.float32).view(1, H, dk, dv)
        else:
            kw["o"] = d["v" if over == "all" else over]
        args = (d["q"], d["k"], d["v"], d["beta"], d["log_alpha"])
        o, ht = (G.gdn_chunk_fwd_save(*args, **kw)[:2] if save else G.gdn_chunk_fwd(*args, **kw))
        torch.cuda.synchronize()
        assert torch.equal(o, want_o) and torch.equal(ht, want_ht), (over, save)


@pytest.mark.parametrize("dk,dv,H,last", [(256, 512, 32, 1), (256, 512, 32, 4), (128, 128, 128, 1),
                                          (128, 128, 128, 32)])
def test_shapes_agree_around_their_line(G, dk, dv, H, last):
    """One sequence with as many heads as fill the chip once, and the same
    heads beside ``last`` more of them: the passes of other shapes, the same
    bits.  Also packed, where the lines lie elsewhere: a short second sequence."""
    T = 330
    inp = problem(dk, dv, 1, H + last, T, seed=35, h0_std=0.05, backward=True)
    few = {n: x[:, :H].contiguous() if n in ("h0", "dht") else x[:, :, :H].contiguous()
           for n, x in inp.items() if isinstance(x, torch.Tensor)}
    say("line", dk, dv, H, last)
    one, more = training_step(G, to_dev(few)), training_step(G, to_dev(inp))
    cu = torch.tensor([0, 200, T], dtype=torch.int32)
    pack = dict(few, cu_seqlens=cu, h0=few["h0"].repeat(2, 1, 1, 1), dht=few["dht"].repeat(2, 1, 1, 1))
    for n in one:
        cut = more[n][:, :H] if n in ("ht", "dh0") else more[n][:, :, :H]
        assert torch.equal(one[n], cut), n
    packed = training_step(G, to_dev(pack))
    alone = G.gdn_chunk_fwd(*(to_dev(few)[n][:, :200].contiguous()
                              for n in ("q", "k", "v", "beta", "log_alpha")), h0=few["h0"].cuda())
    torch.cuda.synchronize()
    assert torch.equal(packed["o"][:, :200], alone[0]) and torch.equal(packed["ht"][:1], alone[1])
