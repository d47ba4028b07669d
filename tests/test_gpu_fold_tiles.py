"""Folds at the edges of the sort's and the segment passes' tiles (GPU):
entry counts around 1,024, 2,048 and 8,192, key widths of one to eight digits,
values of 1, 4 and 8 bytes, segments inside a tile, across tiles and over the
whole input, dropped segments, gaps between rows and permuted modes.  Sums are
formed in 64 bits in input order and rounded once on both sides, so outputs
are equal bit for bit."""

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


def same(ctx, semiring, dtype, r, c, v, m, n):
    got = gpu_fold(ctx, semiring, dtype, r, c, v, m, n)
    exp = oracle.fold(semiring, dtype, r, c, v, m, n)
    rp, col, val = got.to_host()
    assert np.array_equal(rp, exp.rowptr) and np.array_equal(col, exp.col)
    assert np.array_equal(val, exp.val)


SIZES = [1, 2, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049, 8191, 8192, 8193, 16384, 24577, 300007]


@pytest.mark.parametrize("nnz", SIZES)
@pytest.mark.parametrize("semiring,dtype", [("plus_times", "f64"), ("plus_times", "f32"), ("min_plus", "i32"),
                                            ("or_and", "bool")])
def test_entry_counts(ctx, semiring, dtype, nnz):
    say("fold entries", semiring, dtype, nnz)
    rng = np.random.default_rng(nnz)
    for m, n in ((1, 1), (13, 19), (1000, 70), (5, 1 << 30), (1 << 16, 1 << 30)):
        if m * nnz > 1 << 33:
            m = 300
        r, c = rng.integers(0, m, nnz), rng.integers(0, n, nnz)
        same(ctx, semiring, dtype, r, c, values(semiring, dtype, nnz, 3, nnz), m, n)


@pytest.mark.parametrize("nnz", [4095, 8192, 40000])
def test_long_segments_and_drops(ctx, nnz):
    say("fold segments", nnz)
    rng = np.random.default_rng(nnz)
    m, n = 3000, 50
    # segments of about a third of a tile, of several tiles, and single ones
    r = np.where(rng.random(nnz) < 0.7, 1500, np.where(rng.random(nnz) < 0.8, 17, rng.integers(0, m, nnz)))
    c = np.where(r == 1500, 7, rng.integers(0, n, nnz))
    v = values("plus_times", "f32", nnz, 9)
    same(ctx, "plus_times", "f32", r, c, v, m, n)
    # entries that cancel in pairs, and entries equal to the identity
    v = np.tile(np.array([1.5, -1.5]), (nnz + 1) // 2)[:nnz]
    r2, c2 = np.repeat(r, 2)[:nnz], np.repeat(c, 2)[:nnz]
    v[::7] = 0.0
    v[1::14] = 0.0
    same(ctx, "plus_times", "f64", r2, c2, v, m, n)
    same(ctx, "plus_times", "f64", r2, c2, np.zeros(nnz), m, n)


def test_modes_permuted(ctx):
    say("fold modes")
    rng = np.random.default_rng(5)
    dims, nnz = (7, 1, 33, 5), 9000
    idx = [rng.integers(0, d, nnz) for d in dims]
    v = values("plus_times", "f64", nnz, 4)
    key = np.ravel_multi_index(idx, dims)
    coo = srtc.COO(torch.as_tensor(key, device="cuda"), torch.as_tensor(v, device="cuda"), dims)
    for rows, cols in (("ca", "db"), ("d", "abc"), ("abcd"[:2], "cd"), ("bdc", "a")):
        got = ctx.fold("plus_times", coo, "abcd", rows, cols)
        at = {ch: q for q, ch in enumerate("abcd")}
        ravel = lambda ls: (np.ravel_multi_index([idx[at[x]] for x in ls], [dims[at[x]] for x in ls]),
                            int(np.prod([dims[at[x]] for x in ls])))
        (r, m), (c, n) = ravel(rows), ravel(cols)
        exp = oracle.fold("plus_times", "f64", r, c, v, m, n)
        rp, col, val = got.to_host()
        assert np.array_equal(rp, exp.rowptr) and np.array_equal(col, exp.col) and np.array_equal(val, exp.val)
