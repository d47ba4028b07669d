"""Batches of small dense products (GPU): sizes around the line between a
thread per entry and a tile per product, and their time against one product of
as many terms."""

import time

import pytest
import torch

import paper_1512_00066_amd as srtc
from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return srtc.Context(0)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("z,m,n,k", [(257, 1, 1, 1), (300, 3, 3, 3), (1000, 8, 8, 8), (300, 2, 64, 5), (300, 64, 2, 5),
                                     (300, 2, 65, 5), (260, 16, 16, 256), (260, 16, 16, 257), (260, 24, 24, 24),
                                     (260, 25, 25, 25), (260, 36, 36, 33), (256, 8, 8, 8), (70000, 2, 3, 4)])
def test_small_batches(ctx, dtype, z, m, n, k):
    say("gemm batch", dtype, z, m, n, k)
    g = torch.Generator().manual_seed(z + m + n + k)
    a, b, c = (torch.rand(s, generator=g, dtype=torch.float64).to(dtype) for s in ((z, m, k), (z, k, n), (z, m, n)))
    exp = torch.matmul(a.double(), b.double())
    # positive terms: fp64 sums of k lose at most k 2^-53 on either side; fp32
    # ones are exact products, at most 128 summed in fp32, and round once
    tol = 2 * (k + 1) * 2.0**-53 if dtype == torch.float64 else 130 * 2.0**-24
    for accumulate in (False, True):
        C = c.cuda()
        ctx.contract("plus_times", "zik", a.cuda(), "zkj", b.cuda(), "zij", C=C, accumulate=accumulate)
        ref = exp + c.double() if accumulate else exp
        assert torch.all((C.cpu().double() - ref).abs() <= tol * ref)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_many_small_products_are_one_short_launch(ctx, dtype):
    """10,000 of 8 x 8 x 8 move 15 MB; 10,000 x 8 x 8 moves a third of it and is
    a launch of no length either."""
    say("gemm batch time", dtype)
    best = []
    for shape in ((10000, 8, 8, 8), (1, 10000, 8, 8)):
        z, m, n, k = shape
        A, B = torch.rand(z, m, k, device="cuda", dtype=dtype), torch.rand(z, k, n, device="cuda", dtype=dtype)
        C = torch.empty(z, m, n, device="cuda", dtype=dtype)
        one = []
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(40):
                ctx.contract("plus_times", "zik", A, "zkj", B, "zij", C=C)
            torch.cuda.synchronize()
            one.append(time.perf_counter() - t)
        best.append(min(one))
    assert best[0] <= 3 * best[1], best
