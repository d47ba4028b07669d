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


@pytest.mark.parametrize("m", [1000, 3000])
def test_narrow_products_of_split_rows(ctx, m):
    """One column: 100 nonzeros a row are four items and a combination, 32 are
    one item; the items run side by side and the combination is one more short
    launch."""
    say("narrow split rows", m)
    whole, split = (product_time(ctx, uniform(m, 2000, d, m), 1) for d in (32, 100))
    assert split <= 2.5 * whole, (whole, split)


@pytest.mark.parametrize("width", [1, 2, 3, 8, 16, 31, 32, 33, 64])
@pytest.mark.parametrize("m", [5, 700, 9000])
def test_split_rows_of_every_share(ctx, m, width):
    """Runs of split and whole rows of all lengths, combined by groups of 1 to
    64 lanes: integer values, so sums are equal whatever their order."""
    say("split rows", m, width)
    g = torch.Generator().manual_seed(m + width)
    k = 900
    ln = torch.randint(0, 40, (m,), generator=g)
    ln[torch.rand(m, generator=g) < 0.4] = 33
    ln[m // 2: m // 2 + 3] = torch.tensor([64, 900, 257])[: len(ln[m // 2: m // 2 + 3])]
    rp = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(ln, 0)])
    col = torch.cat([torch.randperm(k, generator=g)[:int(x)].sort().values for x in ln])
    val = torch.randint(1, 9, (int(rp[-1]),), generator=g).double()
    X = torch.randint(1, 9, (k, width), generator=g).double()
    dense = torch.zeros((m, k), dtype=torch.float64)
    dense[torch.repeat_interleave(torch.arange(m), ln), col] = val
    A = srtc.CSR(rp.cuda(), col.int().cuda(), val.cuda(), (m, k))
    Y = torch.empty((m, width), dtype=torch.float64, device="cuda")
    ctx.contract("plus_times", "ik", A, "kj", X.cuda(), "ij", C=Y)
    assert torch.equal(Y.cpu(), dense @ X)
    ctx.contract("plus_times", "ik", A, "kj", X.cuda(), "ij", C=Y, accumulate=True)
    assert torch.equal(Y.cpu(), 2 * (dense @ X))
