"""Rows at the edges of the SpGEMM bins (GPU): output counts around every
table size, columns spread over B's range (placed by bucket rank) or
contiguous in a wide matrix (one crowded bucket, sorted instead), numbers of
rows around the one-launch binning's limit, and A rows around the length
from which a whole block counts their products."""

import numpy as np
import pytest

import oracle
import paper_1512_00066_amd as srtc
from gpu_common import check_csr, gpu_fold, say, values

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return srtc.Context(0)


def product(ctx, semiring, dtype, a, b, m, k, n, sorted_rows=True, schedule=0):
    (ar, ac), (br, bc) = a, b
    av, bv = values(semiring, dtype, ar.size, 5, 1), values(semiring, dtype, br.size, 5, 2)
    GA, GB = gpu_fold(ctx, semiring, dtype, ar, ac, av, m, k), gpu_fold(ctx, semiring, dtype, br, bc, bv, k, n)
    exp = oracle.spgemm(semiring, dtype, oracle.fold(semiring, dtype, ar, ac, av, m, k),
                        oracle.fold(semiring, dtype, br, bc, bv, k, n))
    got = ctx.contract(semiring, "ik", GA, "kj", GB, "ij", schedule=schedule, sorted=sorted_rows)
    if not sorted_rows:
        rp, col, val = got.to_host()
        for r in range(m):
            o = np.argsort(col[rp[r]:rp[r + 1]], kind="stable") + rp[r]
            col[rp[r]:rp[r + 1]], val[rp[r]:rp[r + 1]] = col[o], val[o]
        got = srtc.csr_from_host(rp, col, val, (m, n))
    check_csr(got, exp, semiring, dtype)


EDGES = [1, 31, 32, 33, 64, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097]


@pytest.mark.parametrize("sorted_rows", [True, False])
@pytest.mark.parametrize("spread", ["spread", "contiguous", "mixed"])
@pytest.mark.parametrize("semiring,dtype", [("min_plus", "i32"), ("plus_times", "f64"), ("or_and", "bool")])
def test_output_counts_at_table_edges(ctx, semiring, dtype, spread, sorted_rows):
    say("bin edges", semiring, dtype, spread, sorted_rows)
    n = 131101
    rng = np.random.default_rng(17)
    br, bc = [], []
    for k, ln in enumerate(EDGES):
        if spread == "spread":
            cols = rng.choice(n, ln, replace=False)
        elif spread == "contiguous":
            cols = (n - ln) // 2 + np.arange(ln)
        else:  # half in one stretch, the last column, the rest anywhere
            cols = np.unique(np.concatenate([np.arange(ln // 2), rng.choice(n, ln - ln // 2), [n - 1]]))
        br.append(np.full(cols.size, k))
        bc.append(cols)
    # rows of A: one B row alone, and one B row met twice by way of a copy
    kk = len(EDGES)
    br2 = br + [x + kk for x in br]
    bc2 = bc + bc
    ar = np.concatenate([np.arange(kk), kk + np.repeat(np.arange(kk), 2)])
    ac = np.concatenate([np.arange(kk), np.stack([np.arange(kk), np.arange(kk) + kk], 1).reshape(-1)])
    product(ctx, semiring, dtype, (ar, ac), (np.concatenate(br2), np.concatenate(bc2)), 2 * kk, 2 * kk, n, sorted_rows)


@pytest.mark.parametrize("m", [1, 255, 257, 4095, 4096, 4097, 262145])
def test_row_counts_of_the_binning(ctx, m):
    say("binning rows", m)
    rng = np.random.default_rng(m)
    k, n = 300, 5000
    deg = rng.integers(0, 4, m)
    ar = np.repeat(np.arange(m), deg)
    ac = rng.integers(0, k, ar.size)
    bl = np.concatenate([np.zeros(60, np.int64), rng.integers(1, 40, 200), rng.integers(40, 700, 40)])
    br = np.repeat(np.arange(k), bl)
    bc = rng.integers(0, n, br.size)
    if m > 100000:  # most rows empty: the lists still hold every other one
        keep = rng.random(ar.size) < 0.05
        ar, ac = ar[keep], ac[keep]
    product(ctx, "min_plus", "i32", (ar, ac), (br, bc), m, k, n)


@pytest.mark.parametrize("length", [15, 16, 17, 64, 255, 256, 257, 511, 1281, 5000])
def test_row_products_of_long_rows(ctx, length):
    say("row products", length)
    rng = np.random.default_rng(length)
    m, k, n = 37, 6000, 800
    lens = np.where(np.arange(m) % 5 == 2, length, rng.integers(0, 6, m))
    ar = np.repeat(np.arange(m), lens)
    ac = np.concatenate([rng.choice(k, x, replace=False) for x in lens])
    br = np.repeat(np.arange(k), rng.integers(0, 4, k))
    bc = rng.integers(0, n, br.size)
    one = np.ones(max(ar.size, br.size), np.int32)
    A = gpu_fold(ctx, "min_plus", "i32", ar, ac, one[:ar.size], m, k)
    B = gpu_fold(ctx, "min_plus", "i32", br, bc, one[:br.size], k, n)
    got = ctx.features("min_plus", A, B)
    exp = oracle.features("min_plus", oracle.fold("min_plus", "i32", ar, ac, one[:ar.size], m, k),
                          oracle.fold("min_plus", "i32", br, bc, one[:br.size], k, n))
    # product histogram: whole-number counts over rows, exact
    assert np.array_equal(got[10:20], np.asarray(exp, np.float32)[10:20])
    # log2 of the product total and of the largest row's products: the same
    # whole numbers under the same fp32 rounding of a log2
    np.testing.assert_allclose(got[[23, 25]], np.asarray(exp, np.float32)[[23, 25]], rtol=2e-7)
    product(ctx, "plus_times", "f64", (ar, ac), (br, bc), m, k, n)
