"""The timing record's launch names lead to kernels that exist: every key that
profiling.kernel_key() forms of a name the library gives to a launch is a
kernel of the built library, and every such name has a work model in bench.py
(CPU only)."""
import os
import re

import pytest

from paper_2412_06464_amd import gdn, profiling
from tests.test_bench_models import bench, wl  # noqa: F401 (fixture)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DIMS = [(64, 64), (128, 128), (256, 512)]
HELPERS = {"k_chunk_table", "k_copy", "k_conv_bwd_qk"}  # no template, or two kernels


@pytest.fixture(scope="module")
def built():
    """Keys of the kernels in libgdn.so, from its kernels' symbol names."""
    if not os.path.exists(gdn.LIB_PATH):
        from paper_2412_06464_amd import build
        build.build()
    lib = open(gdn.LIB_PATH, "rb").read()
    names = {n.decode() for n in re.findall(rb"_ZN3gdn\d+k_[A-Za-z0-9_]+E(?=\0)", lib)}
    assert names
    return {profiling.kernel_key_of(n) for n in names}


def launch_names():
    """Every name gdn_launch.hip gives to a launch."""
    src = open(os.path.join(ROOT, "paper_2412_06464_amd", "csrc", "gdn_launch.hip")).read()
    names = set(re.findall(r'"(k_[a-z_]+)"', src))
    assert {"k_prep", "k_fwd_chain_save", "k_bwd_chain", "k_prep_small_save_block"} <= names
    return sorted(names)


@pytest.mark.parametrize("name", launch_names())
def test_every_launch_name_has_its_kernels(built, name):
    if name in HELPERS:
        return
    chain = "chain" in name or "small" in name
    block = "block" in name or name == "k_conv_bwd"
    for dtype in ("bf16",) if chain or block else ("bf16", "f32"):
        for dk, dv in DIMS:
            for call in ("fwd", "bwd"):
                if call == "bwd" and "prep" in name and ("save" in name or block):
                    continue  # the backward's prep neither saves nor runs the prologue
                key = profiling.kernel_key(call + ":" + name, dtype, dk, dv)
                if key.endswith(","):
                    assert any(k.startswith(key) for k in built), key
                else:
                    assert key in built, key


def test_find_kernel():
    rec = {"k_fwd_chain<256,512,2,2,4>": 1, "k_fwd_chain<256,512,0,2,4>": 2, "k_copy": 3}
    key = profiling.kernel_key("fwd:k_fwd_chain_save", "bf16", 256, 512)
    assert profiling.find_kernel(rec, key) == 1
    assert profiling.find_kernel(rec, "k_copy") == 3
    assert profiling.find_kernel(rec, "k_fwd_chain<128,128,2,") is None
    rec["k_fwd_chain<256,512,2,1,4>"] = 4  # two shapes in one run: which is not known
    assert profiling.find_kernel(rec, key) is None


@pytest.mark.parametrize("dk,dv", DIMS)
def test_chain_step_models(bench, dk, dv):  # noqa: F811
    """The launches of a saved training step by the chain passes: the path's
    FLOP without W~ (2 C dk a token-head), and the path's bytes with what a
    second launch reads again: k and q by the saving pass, k, q and dO by the
    reverse pass."""
    w = wl(dk, dv, "bf16", True, 3)
    th, nseq, e = 5000, 4, 2
    m = bench.kernel_models(w, th, nseq * w.H, True)
    names = ("k_prep_small_save", "k_fwd_chain_save", "k_bwd_chain", "k_grad")
    flop = sum(m[k][1] for k in names)
    assert flop == pytest.approx(bench.path_flops(w, th) - 2 * 64 * dk * th, rel=1e-12)
    again = 2 * dk + 2 * dk + dv
    assert sum(m[k][0] for k in names) == (bench.path_bytes(w, th, nseq, True, saved=True)
                                           + th * again * e)
    for name in launch_names():
        assert name in bench.fused_models(w, th, nseq * w.H, True) or name == "k_recurrent", name
