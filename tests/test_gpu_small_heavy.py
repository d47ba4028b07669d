"""Products of few rows and columns but many products (GPU): dense rows of
unequal weight, more and fewer than there are compute units, against long and
short rows of B; and the time of their counting pass."""

import numpy as np
import pytest
import torch

import oracle
import paper_1512_00066_amd as srtc
from gpu_common import check_csr, gpu_fold, say, values
from gpu_profile import best_times

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return srtc.Context(0)


@pytest.mark.parametrize("semiring,dtype", [("plus_times", "f64"), ("min_plus", "i32"), ("or_and", "bool")])
@pytest.mark.parametrize("m,k,n,db", [(600, 500, 16384, 100), (3, 4000, 9000, 300), (40, 30000, 16000, 3),
                                      (700, 20000, 12000, 2), (1, 513, 5000, 19), (2, 1025, 5000, 21)])
def test_unequal_dense_rows(ctx, semiring, dtype, m, k, n, db):
    say("small heavy", semiring, dtype, m, k, n, db)
    rng = np.random.default_rng(m + k)
    la = np.minimum(k, (k * rng.random(m) ** 4).astype(np.int64) + 1)
    la[m // 2] = k
    if la.sum() * db > 4_000_000:  # (the oracle's time)
        la = np.maximum(1, la * 4_000_000 // (la.sum() * db))
        la[m // 2] = k
    lb = rng.integers(max(1, db - 3), db + 4, k)
    ar, br = np.repeat(np.arange(m), la), np.repeat(np.arange(k), lb)
    ac = np.concatenate([rng.choice(k, x, replace=False) for x in la])
    bc = rng.integers(0, n, br.size)
    av, bv = values(semiring, dtype, ar.size, 5, m), values(semiring, dtype, br.size, 6, n)
    A, B = gpu_fold(ctx, semiring, dtype, ar, ac, av, m, k), gpu_fold(ctx, semiring, dtype, br, bc, bv, k, n)
    exp = oracle.spgemm(semiring, dtype, oracle.fold(semiring, dtype, ar, ac, av, m, k),
                        oracle.fold(semiring, dtype, br, bc, bv, k, n))
    for schedule in (0, 2, 3):
        check_csr(ctx.contract(semiring, "ik", A, "kj", B, "ij", schedule=schedule), exp, semiring, dtype)


def test_counting_costs_less_than_multiplying(ctx):
    """One row of 4,096 entries against rows of 400: the counting pass reads
    half the bytes of the numeric one and sets a bit where that adds."""
    say("small heavy time")
    g = torch.Generator().manual_seed(4)
    k = n = 4096
    col = torch.stack([torch.randperm(n, generator=g)[:400].sort().values for _ in range(k)]).reshape(-1).int()
    val = torch.randint(1, 50, (k * 400,), generator=g).int()
    B = srtc.CSR(torch.arange(k + 1).mul(400).cuda(), col.cuda(), val.cuda(), (k, n))
    A = srtc.CSR(torch.tensor([0, k]).cuda(), torch.arange(k).int().cuda(), val[:k].cuda(), (1, k))
    best = best_times(ctx, lambda: ctx.contract("min_plus", "ik", A, "kj", B, "ij"))
    numeric = sum(ms for name, ms in best.items() if name.startswith("spgemm.numeric"))
    assert best["spgemm.symbolic.small"] <= 0.8 * numeric, best
