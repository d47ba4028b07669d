"""Small sparse x dense products (GPU): their times, by the library's events,
against those of like products that take another kernel."""

import pytest
import torch

import paper_1512_00066_amd as srtc
from gpu_common import say
from gpu_profile import best_times

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return srtc.Context(0)


def uniform(m, k, d, seed):
    """m x k CSR of d random nonzeros a row."""
    g = torch.Generator().manual_seed(seed)
    col = torch.stack([torch.randperm(k, generator=g)[:d].sort().values for _ in range(m)]).reshape(-1)
    val = torch.rand(m * d, generator=g, dtype=torch.float64)
    return srtc.CSR(torch.arange(m + 1).mul(d).cuda(), col.int().cuda(), val.cuda(), (m, k))


def product_time(ctx, A, width):
    X = torch.ones((A.dims[1], width), dtype=torch.float64, device="cuda")
    Y = torch.empty((A.dims[0], width), dtype=torch.float64, device="cuda")
    call = lambda: ctx.contract("plus_times", "ik", A, "kj", X, "ij", C=Y)
    call()
    return best_times(ctx, call, 10)["spmm.product"]


@pytest.mark.parametrize("m", [300, 1000, 3000])
def test_wide_products_of_few_short_rows(ctx, m):
    """64 columns in units of consecutive nonzeros, 32 in items of a row each:
    twice the columns, and both fit the chip at once."""
    say("small wide product", m)
    A = uniform(m, 2000, 10, m)
    narrow, wide = product_time(ctx, A, 32), product_time(ctx, A, 64)
    assert wide <= 2.5 * narrow, (narrow, wide)
