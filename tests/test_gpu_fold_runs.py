"""Folds of many entries to few outputs (GPU): runs of one key around the
lengths that the segment passes bring in at a time, and their time against a
fold of as many entries to as many outputs."""

import time

import numpy as np
import pytest
import torch

import oracle
import paper_1512_00066_amd as srtc
from gpu_common import gpu_fold, say, values

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return srtc.Context(0)


@pytest.mark.parametrize("lead", [0, 1, 2047, 2048, 2050])
@pytest.mark.parametrize("run", [2, 9, 64, 2047, 2048, 2049, 4095, 4096, 4097, 6144, 6145])
@pytest.mark.parametrize("semiring,dtype", [("plus_times", "f64"), ("plus_times", "f32"), ("min_plus", "i32"),
                                            ("or_and", "bool")])
def test_runs_across_tiles(ctx, semiring, dtype, run, lead):
    """`lead` single entries, a run, and single entries: the run starts and ends
    anywhere in a tile, and at the input's end (equal bit for bit: sums are in
    input order in 64 bits on both sides)."""
    say("fold run", semiring, dtype, run, lead)
    rng = np.random.default_rng(run + lead)
    for tail in (0, 1, 700):
        c = np.concatenate([np.arange(lead), np.full(run, lead + 1), lead + 2 + np.arange(tail)])
        order = rng.permutation(c.size)
        c, v = c[order], values(semiring, dtype, c.size, run, lead)
        if dtype != "bool":
            v[::11] = oracle.default_add_id(semiring, dtype)  # entries that count as absent
        n = lead + tail + 3
        got = gpu_fold(ctx, semiring, dtype, np.zeros_like(c), c, v, 1, n)
        exp = oracle.fold(semiring, dtype, np.zeros_like(c), c, v, 1, n)
        rp, col, val = got.to_host()
        assert np.array_equal(rp, exp.rowptr) and np.array_equal(col, exp.col) and np.array_equal(val, exp.val)


def test_a_run_that_cancels_is_dropped(ctx):
    say("fold run dropped")
    v = np.tile([1.0, -1.0], 4000)
    c = np.full(8000, 3)
    got = gpu_fold(ctx, "plus_times", "f64", np.zeros_like(c), c, v, 1, 9)
    assert got.nnz == 0 and torch.equal(got.rowptr.cpu(), torch.tensor([0, 0]))
    v[5] = 2.0
    got = gpu_fold(ctx, "plus_times", "f64", np.zeros_like(c), c, v, 1, 9)
    assert got.col.tolist() == [3] and got.val.tolist() == [3.0]


def test_few_outputs_cost_about_what_many_do(ctx):
    """2^22 entries, 300 to an output, against one to an output: the sort is the
    same, and a segment pass may at most wait for 300 additions in a row."""
    say("fold time of runs")
    n, best = 1 << 22, {}
    g = torch.Generator().manual_seed(2)
    v = torch.rand(n, generator=g).cuda()
    for per in (1, 300):
        keys = torch.randint(0, n // per, (n,), generator=g).cuda()
        coo = srtc.COO(keys, v, (n // per, 1))
        for _ in range(8):
            torch.cuda.synchronize()
            t = time.perf_counter()
            ctx.fold("plus_times", coo, "ab", "a", "b")
            torch.cuda.synchronize()
            best[per] = min(best.get(per, 1.0), time.perf_counter() - t)
    assert best[300] <= 2.6 * best[1], best
