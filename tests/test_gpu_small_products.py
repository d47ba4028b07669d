"""Small products (GPU): the shapes around the limits under which all rows'
output counts are formed in one launch from column bitmaps and the row
pointers and bins in another: 4,096 rows and 16,384 columns."""

import numpy as np
import pytest

import oracle
import paper_1512_00066_amd as srtc
from gpu_common import check_csr, gpu_fold, say, values

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return srtc.Context(0)


def operands(semiring, dtype, m, k, n, da, db, seed, hub):
    rng = np.random.default_rng(seed)
    la = rng.integers(0, 2 * da + 1, m)
    lb = rng.integers(0, 2 * db + 1, k)
    if hub:  # one long row of A, one of B that covers every column
        la[m // 2] = min(k, 3000)
        lb[k // 3] = n
    ar, br = np.repeat(np.arange(m), la), np.repeat(np.arange(k), lb)
    ac = np.concatenate([rng.integers(0, k, x) for x in la] + [np.zeros(0, np.int64)])
    bc = np.concatenate([np.arange(n) if x == n else rng.integers(0, n, x) for x in lb])
    return (ar, ac, values(semiring, dtype, ar.size, seed, 1)), (br, bc, values(semiring, dtype, br.size, seed, 2))


@pytest.mark.parametrize("m,k,n", [(1, 1, 1), (3, 5, 31), (64, 64, 32), (65, 7, 33), (1023, 300, 4097),
                                   (1025, 300, 16384), (1025, 300, 16385), (4095, 500, 1000), (4096, 500, 16383),
                                   (4097, 500, 1000)])
@pytest.mark.parametrize("semiring,dtype", [("min_plus", "i32"), ("plus_times", "f64"), ("or_and", "bool")])
@pytest.mark.parametrize("hub", [False, True])
def test_small_shapes(ctx, semiring, dtype, m, k, n, hub):
    say("small product", semiring, dtype, m, k, n, hub)
    (ar, ac, av), (br, bc, bv) = operands(semiring, dtype, m, k, n, 3, 4, m + n, hub)
    A, B = gpu_fold(ctx, semiring, dtype, ar, ac, av, m, k), gpu_fold(ctx, semiring, dtype, br, bc, bv, k, n)
    exp = oracle.spgemm(semiring, dtype, oracle.fold(semiring, dtype, ar, ac, av, m, k),
                        oracle.fold(semiring, dtype, br, bc, bv, k, n))
    for schedule in (0, 3):
        check_csr(ctx.contract(semiring, "ik", A, "kj", B, "ij", schedule=schedule), exp, semiring, dtype)


def test_small_product_empty_and_cancelled(ctx):
    say("small product empty")
    e = np.zeros(0, np.int64)
    A, B = gpu_fold(ctx, "plus_times", "f64", e, e, np.zeros(0, np.float64), 40, 50), \
        gpu_fold(ctx, "plus_times", "f64", e, e, np.zeros(0, np.float64), 50, 60)
    assert ctx.contract("plus_times", "ik", A, "kj", B, "ij").nnz == 0
    # every row's products cancel in its first output: dropped, rest kept
    m = 700
    ar, ac = np.repeat(np.arange(m), 2), np.tile([0, 1], m)
    av = np.tile(np.array([1, -1], np.float64), m)
    br, bc, bv = np.array([0, 1, 1]), np.array([5, 5, 9]), np.array([3, 3, 4], np.float64)
    A, B = gpu_fold(ctx, "plus_times", "f64", ar, ac, av, m, 2), gpu_fold(ctx, "plus_times", "f64", br, bc, bv, 2, 12)
    rp, col, val = ctx.contract("plus_times", "ik", A, "kj", B, "ij").to_host()
    assert np.array_equal(rp, np.arange(m + 1)) and np.all(col == 9) and np.all(val == -4)


@pytest.mark.parametrize("m", [4097, 5121, 16383, 16384, 16385])
def test_rows_around_the_one_block_scan(ctx, m):
    """Row pointers from the scan in one block (up to 16,384 rows) and from
    the tiled one."""
    say("one-block scan", m)
    (ar, ac, av), (br, bc, bv) = operands("min_plus", "i32", m, 200, 900, 2, 3, m, True)
    A, B = gpu_fold(ctx, "min_plus", "i32", ar, ac, av, m, 200), gpu_fold(ctx, "min_plus", "i32", br, bc, bv, 200, 900)
    exp = oracle.spgemm("min_plus", "i32", oracle.fold("min_plus", "i32", ar, ac, av, m, 200),
                        oracle.fold("min_plus", "i32", br, bc, bv, 200, 900))
    check_csr(ctx.contract("min_plus", "ik", A, "kj", B, "ij"), exp, "min_plus", "i32")
