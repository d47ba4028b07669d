"""Few rows of which one has most of the products (GPU): the dense windows
they take are the wide ones.  Rows of A around the block sizes of the dense
kernels, outputs in one window and over all of them."""

import numpy as np
import pytest

import oracle
import paper_1512_00066_amd as srtc
from gpu_common import check_csr, gpu_fold, say, values

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return srtc.Context(0)


@pytest.mark.parametrize("n", [9000, 70001])
@pytest.mark.parametrize("hub", [500, 513, 1024, 1025, 4000])
@pytest.mark.parametrize("semiring,dtype", [("plus_times", "f64"), ("plus_times", "f32"), ("min_plus", "i32"),
                                            ("or_and", "bool")])
def test_hub_row(ctx, semiring, dtype, hub, n):
    say("hub panel", semiring, dtype, hub, n)
    rng = np.random.default_rng(hub + n)
    m, k, per = 40, 4000, 300
    lens = rng.integers(0, 25, m)
    lens[17] = hub
    ar = np.repeat(np.arange(m), lens)
    ac = np.concatenate([rng.choice(k, x, replace=False) for x in lens])
    br = np.repeat(np.arange(k), per)
    bc = rng.integers(0, n, br.size)
    av, bv = values(semiring, dtype, ar.size, 6, 1), values(semiring, dtype, br.size, 6, 2)
    A, B = gpu_fold(ctx, semiring, dtype, ar, ac, av, m, k), gpu_fold(ctx, semiring, dtype, br, bc, bv, k, n)
    exp = oracle.spgemm(semiring, dtype, oracle.fold(semiring, dtype, ar, ac, av, m, k),
                        oracle.fold(semiring, dtype, br, bc, bv, k, n))
    for schedule in (0, 5):
        check_csr(ctx.contract(semiring, "ik", A, "kj", B, "ij", schedule=schedule), exp, semiring, dtype)
