"""Dense rounds of path doubling at the edges of their 64 x 64 tiles and of
the 32-deep k-tiles (GPU): distances and hop counts equal the oracle's."""

import numpy as np
import pytest
import torch

import oracle
import paper_1512_00066_amd as srtc
from gen import synth
from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 31, 32, 33, 63, 64, 65, 95, 96, 97, 128, 129, 193])
@pytest.mark.parametrize("keep", [1.0, 0.4])
def test_dense_round_edges(n, keep):
    say("apsp tiles", n, keep)
    ctx = srtc.Context(0)
    src, dst, w = synth.dense_graph(n, 11, hi=50)
    sel = np.random.default_rng(n).random(src.size) < keep
    src, dst, w = src[sel], dst[sel], w[sel].astype(np.int32)
    coo = srtc.COO(torch.as_tensor(dst * n + src, device="cuda"), torch.as_tensor(w, device="cuda"), (n, n))
    D, H, rounds = ctx.apsp_tiskin(coo)
    Do, Ho, ro, _ = oracle.apsp_tiskin(oracle.fold("min_plus", "i32", dst, src, w, n, n), inf_value=oracle.INT_INF)
    assert np.array_equal(D.cpu().numpy().astype(np.int64), Do)
    assert np.array_equal(H.cpu().numpy().astype(np.int64), Ho)
    assert rounds == ro
