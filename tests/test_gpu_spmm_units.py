"""Sparse x dense products wider than 32 columns, fixpoint steps and BFS at
the edges of their work units (GPU): runs of empty rows, rows around an
item's length and around the sums' grain, chunk counts around eight, rows
around the length that a whole block takes."""

import numpy as np
import pytest
import torch

import oracle
import paper_1512_00066_amd as srtc
from gpu_common import EXACT, RTOL, TORCH, gpu_fold, say, values

pytestmark = pytest.mark.gpu
INF = oracle.INT_INF


@pytest.fixture(scope="module")
def ctx():
    return srtc.Context(0)


def lengths(rng):
    runs = [[0] * 70, [1] * 130, [63, 64, 65, 0, 0, 127, 128, 129], [255, 256, 257, 511, 512, 513, 0, 1, 1500],
            list(rng.integers(0, 30, 200)), [0] * 64, [2]]
    return np.concatenate([np.asarray(r, np.int64) for r in runs])


def matrix(seed, k):
    rng = np.random.default_rng(seed)
    ln = lengths(rng)
    r = np.repeat(np.arange(ln.size), ln)
    c = np.concatenate([rng.choice(k, x, replace=False) for x in ln]).astype(np.int64)
    return r, c, ln.size


@pytest.mark.parametrize("semiring,dtype", [("plus_times", "f64"), ("plus_times", "f32"), ("min_plus", "i32"),
                                            ("or_and", "bool"), ("max_times", "f64")])
@pytest.mark.parametrize("width", [33, 64, 65, 129, 448, 512, 513, 600, 1024])
def test_wide_products(ctx, semiring, dtype, width):
    say("spmm units", semiring, dtype, width)
    k = 1600
    r, c, m = matrix(width, k)
    v = values(semiring, dtype, r.size, 31, 1)
    A = gpu_fold(ctx, semiring, dtype, r, c, v, m, k)
    O = oracle.fold(semiring, dtype, r, c, v, m, k)
    x = values(semiring, dtype, k * width, 31, 2).reshape(k, width).copy()
    idv = oracle.default_add_id(semiring, dtype)
    x[::7, ::3] = idv  # absent entries
    X = torch.as_tensor(x, device="cuda")
    Y = torch.empty((m, width), dtype=TORCH[dtype], device="cuda")
    ref = oracle.spmm(semiring, dtype, O, x)[0]

    def check(got, exp):
        got = got.cpu().numpy()
        if (semiring, dtype) in EXACT:
            assert np.array_equal(got, exp.astype(got.dtype))
        else:
            assert np.all(np.abs(got.astype(np.float64) - exp) <= RTOL[(semiring, dtype)] * np.abs(exp))

    ctx.contract(semiring, "ik", A, "kj", X, "ij", C=Y)
    check(Y, ref)
    # the fixed-buffer form runs the same sums
    Z = torch.empty_like(Y)
    ctx.contract_noalloc(semiring, "ik", A, "kj", X, "ij", Z)
    assert torch.equal(Y, Z)
    if semiring == "plus_times":
        ctx.contract(semiring, "ik", A, "kj", X, "ij", C=Y, accumulate=True)
        check(Y, 2 * ref)


@pytest.mark.parametrize("changed", [False, True])
@pytest.mark.parametrize("nsrc", [40, 64, 100, 520])
def test_fixpoint_wide(ctx, nsrc, changed):
    say("fixpoint units", nsrc, changed)
    n = 1600
    r, c, _ = matrix(3, n)
    w = values("min_plus", "i32", r.size, 6)
    A = gpu_fold(ctx, "min_plus", "i32", r, c, w, n, n)
    O = oracle.fold("min_plus", "i32", r, c, w, n, n)
    P0 = np.full((n, nsrc), INF, np.int32)
    P0[np.arange(nsrc), np.arange(nsrc)] = 0
    X = torch.as_tensor(P0, device="cuda")
    it = ctx.fixpoint("min_plus", A, X, changed_rows_only=changed)
    exp, steps = oracle.bellman_ford("min_plus", "i32", O, P0)[:2]
    assert it == steps and np.array_equal(X.cpu().numpy(), exp)


@pytest.mark.parametrize("nsrc", [1, 17, 64])
def test_bfs_row_lengths(ctx, nsrc):
    say("bfs row lengths", nsrc)
    rng = np.random.default_rng(nsrc)
    n = 9001
    ln = rng.integers(0, 4, n)
    ln[[5, 6, 7, 8, 9, 4000, 9000]] = [511, 512, 513, 1537, 8000, 5000, 600]
    r = np.repeat(np.arange(n), ln)
    c = np.concatenate([rng.choice(n, x, replace=False) for x in ln]).astype(np.int64)
    one = np.ones(r.size, np.uint8)
    A = gpu_fold(ctx, "or_and", "bool", r, c, one, n, n)
    O = oracle.fold("or_and", "bool", r, c, one, n, n)
    src = rng.choice(n, nsrc, replace=False)
    levels, depth = ctx.bfs_levels(A, src)
    exp = np.asarray(oracle.bfs_levels(O, src))
    assert np.array_equal(levels.cpu().numpy(), exp.reshape(levels.shape)) and depth == exp.max()
