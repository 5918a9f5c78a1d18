"""The short convolution's backward and the chunk table at the edges of their tiles.

The backward hands du of a wave's first three rows to the wave before it, and
takes the rows after a full chunk from the next one: lengths around 16 rows (a
wave), 8 (a pass) and 64 (a chunk), each alone in a packed batch, against the
fp64 oracle (same metric and bar as the parity tests).  The chunk table is
written by one workgroup per 256 chunks that scans 256 sequences at a time:
counts of sequences and chunks around 256, with empty sequences.
"""
import numpy as np
import pytest
import torch

from paper_2412_06464_amd.inputs import make_block_inputs
from tests.test_gpu_block import TOL, G, blk, check_conv  # noqa: F401 (fixtures)

pytestmark = pytest.mark.gpu

EDGES = [1, 3, 8, 9, 15, 16, 17, 19, 24, 25, 47, 48, 49, 51, 56, 57, 63, 64, 65, 66, 67, 68, 80,
         128, 130]


@pytest.mark.parametrize("dtype,dk,dv,dim,l2,W", [
    ("f32", 64, 64, 64, True, 4),
    ("bf16", 128, 128, 128, True, 4),
    ("bf16", 256, 512, 256, True, 3),
    ("bf16", 256, 512, 512, False, 4),
])
def test_conv_backward_edges(G, blk, dtype, dk, dv, dim, l2, W):  # noqa: F811
    cu = torch.tensor(np.concatenate([[0], np.cumsum(EDGES)]), dtype=torch.int32)
    inp = make_block_inputs(1, int(cu[-1]), 2, dk, dv, dtype, seed=31, width=W, cu_seqlens=cu)
    x, w, dy = ((inp["xk"], inp["wk"], inp["dk"]) if dim == dk else
                (inp["xv"], inp["wv"], inp["dv"]))
    check_conv(G, blk, x, w, dy, l2, TOL[dtype], "conv_edges_%s_%d" % (dtype, dim), cu=cu)


@pytest.mark.parametrize("lens", [
    [0] * 300 + [70],                          # the first group of 256 holds no chunk
    [64] * 256 + [0] * 3,                      # exactly 256 of each, then empty ones
    [1, 0] * 200 + [65, 64 * 300 + 1, 0, 3],   # 404 sequences, one over more than 256 chunks
], ids=["empties_first", "even_256", "mixed"])
def test_chunk_table_edges(G, blk, lens):  # noqa: F811
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32)
    inp = make_block_inputs(1, int(cu[-1]), 1, 64, 64, "f32", seed=32, width=4, cu_seqlens=cu)
    check_conv(G, blk, inp["xk"], inp["wk"], inp["dk"], True, TOL["f32"], "table", cu=cu)
