"""Dense (+,x) products at the edges of the matrix-core tiles (GPU): sides and
depths around tile and vector sizes, columns no vector divides, both tile
shapes, k split over blocks, batches, signed data."""

import numpy as np
import pytest
import torch

import paper_1512_00066_amd as srtc
from gpu_common import TORCH, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    return srtc.Context(0)


def check(C, a, b, dtype, old=None):
    """|error| against fp64: fp32 sums at most 128 terms in fp32 (one rounding
    per term, relative to the sum of magnitudes) before fp64, then rounds
    once; fp64 at most k + 1 roundings of 2^-53 on either side."""
    a, b = a.astype(np.float64), b.astype(np.float64)
    ref, mag = np.matmul(a, b), np.matmul(np.abs(a), np.abs(b))
    if old is not None:
        ref, mag = ref + old, mag + np.abs(old)
    eps = 128 * 2.0 ** -24 + 2.0 ** -24 if dtype == "f32" else 2 * (a.shape[-1] + 34) * 2.0 ** -53
    err = np.abs(C.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= eps * mag), (err / np.maximum(mag, 1e-300)).max()


def run(ctx, dtype, m, n, k, batch=None):
    rng = np.random.default_rng(m * 7 + n * 3 + k)
    lead = () if batch is None else (batch,)
    a = rng.uniform(-1, 1, lead + (m, k)).astype(np.float64 if dtype == "f64" else np.float32)
    b = rng.uniform(-1, 1, lead + (k, n)).astype(a.dtype)
    C = torch.full(lead + (m, n), float("nan"), dtype=TORCH[dtype], device="cuda")
    ia, ib, ic = ("ik", "kj", "ij") if batch is None else ("zik", "zkj", "zij")
    A, B = torch.as_tensor(a, device="cuda"), torch.as_tensor(b, device="cuda")
    ctx.contract("plus_times", ia, A, ib, B, ic, C=C)
    check(C, a, b, dtype)
    old = C.cpu().numpy().astype(np.float64)
    ctx.contract("plus_times", ia, A, ib, B, ic, C=C, accumulate=True)
    check(C, a, b, dtype, old)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 64, 65, 66, 67, 130])
def test_sides(ctx, dtype, n):
    say("gemm sides", dtype, n)
    for m in (1, 31, 64, 65):
        run(ctx, dtype, m, n, 50)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("k", [1, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 223, 257])
def test_depths(ctx, dtype, k):
    say("gemm depths", dtype, k)
    run(ctx, dtype, 70, 66, k)
    run(ctx, dtype, 65, 67, k)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("m,n,k", [(70, 90, 5000), (64, 64, 4097), (33, 129, 2500), (1, 4, 20000), (4000, 3, 900),
                                   (300, 301, 1031)])
def test_split_depth(ctx, dtype, m, n, k):
    say("gemm split", dtype, m, n, k)
    run(ctx, dtype, m, n, k)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("m,n,k", [(4096, 4096, 37), (4090, 4099, 70), (2048, 2047, 129)])
def test_large_tile(ctx, dtype, m, n, k):
    say("gemm large tile", dtype, m, n, k)
    run(ctx, dtype, m, n, k)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("batch,m,n,k", [(5, 17, 19, 23), (3, 64, 65, 1500), (7, 100, 2, 300), (40, 130, 130, 64)])
def test_batches(ctx, dtype, batch, m, n, k):
    say("gemm batches", dtype, batch, m, n, k)
    run(ctx, dtype, m, n, k, batch)


def test_in_a_captured_graph(ctx):
    """A product that would split k allocates nothing under capture and gives
    the same bits on every replay."""
    a = torch.rand((70, 5000), dtype=torch.float64, device="cuda")
    b = torch.rand((5000, 90), dtype=torch.float64, device="cuda")
    C = torch.zeros((70, 90), dtype=torch.float64, device="cuda")
    ctx.contract("plus_times", "ik", a, "kj", b, "ij", C=C)
    torch.cuda.synchronize()
    before = ctx.allocations
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.contract("plus_times", "ik", a, "kj", b, "ij", C=C)
    assert ctx.allocations == before
    ref = a.cpu().numpy() @ b.cpu().numpy()
    first = None
    for _ in range(3):
        C.zero_()
        g.replay()
        torch.cuda.synchronize()
        got = C.cpu().numpy()
        assert np.all(np.abs(got - ref) <= 1e-12 * np.abs(ref))
        first = got if first is None else first
        assert np.array_equal(got, first)
