"""Masked contraction at the edges of its chunks and queues (GPU): mask rows
around the chunk length, masks that every product hits, that none hits and
that columns share filter bits with, A rows around a block, B rows of one
entry and of thousands."""

import numpy as np
import pytest

import oracle
import paper_1512_00066_amd as srtc
from gpu_common import check_csr, gpu_fold, say, values

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return srtc.Context(0)


@pytest.mark.parametrize("semiring,dtype", [("plus_times", "f64"), ("plus_times", "f32"), ("min_plus", "i32"),
                                            ("or_and", "bool"), ("max_times", "f64")])
@pytest.mark.parametrize("mask", ["full", "none", "half", "aliased"])
def test_masked_edges(ctx, semiring, dtype, mask):
    say("masked edges", semiring, dtype, mask)
    rng = np.random.default_rng(3)
    k, n = 700, 70001
    alen = [0, 1, 2, 63, 64, 255, 256, 257, 600]
    mlen = [0, 1, 2, 63, 64, 65, 1023, 1024, 1025, 2048, 2500]
    rows = [(a, q) for a in alen for q in mlen]
    m = len(rows)
    bl = np.concatenate([[0, 1, 3, 7, 8, 9, 15, 2500, 4000], rng.integers(0, 60, k - 9)])
    br = np.repeat(np.arange(k), bl)
    # B's columns: multiples of 5, so masks can avoid them or share filter bits
    bc = np.concatenate([5 * np.sort(rng.choice(n // 5, x, replace=False)) for x in bl])
    ar = np.concatenate([np.full(a, i) for i, (a, _) in enumerate(rows)])
    ac = np.concatenate([rng.choice(k, a, replace=False) if a else np.zeros(0, np.int64) for a, _ in rows])
    mr, mc = [], []
    for i, (a, q) in enumerate(rows):
        if mask == "full":
            cols = 5 * rng.choice(n // 5, q, replace=False)
        elif mask == "none":
            cols = 5 * rng.choice(n // 5, q, replace=False) + 1
        elif mask == "half":
            cols = rng.choice(n, q, replace=False)
        else:  # the same low bits as B's columns, elsewhere
            cols = np.unique((5 * rng.choice(n // 5, q, replace=False) + 32768) % n)
        mr.append(np.full(cols.size, i))
        mc.append(cols)
    mr, mc = np.concatenate(mr).astype(np.int64), np.concatenate(mc).astype(np.int64)
    av, bv = values(semiring, dtype, ar.size, 8, 1), values(semiring, dtype, br.size, 8, 2)
    one = values(semiring, dtype, mr.size, 8, 3)
    G = [gpu_fold(ctx, semiring, dtype, *x) for x in ((ar, ac, av, m, k), (br, bc, bv, k, n), (mr, mc, one, m, n))]
    O = [oracle.fold(semiring, dtype, *x) for x in ((ar, ac, av, m, k), (br, bc, bv, k, n), (mr, mc, one, m, n))]
    exp = oracle.spgemm_masked(semiring, dtype, *O)
    check_csr(ctx.contract_masked(semiring, "ik", G[0], "kj", G[1], "ij", G[2]), exp, semiring, dtype)
