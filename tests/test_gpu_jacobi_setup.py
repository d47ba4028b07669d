"""The copy of a large Jacobi system's matrix in slices of rows (GPU): what it
costs against an update, which bounds a solve of a few updates, and rows of
every length around the 16 entries that a turn of the copy takes."""

import numpy as np
import pytest
import torch

import oracle
import paper_1512_00066_amd as srtc
from gpu_common import say
from gpu_profile import best_times

pytestmark = pytest.mark.gpu


def banded(n, width):
    """CSR of a band of `width` entries a row, 2 width on the diagonal."""
    c = np.arange(n)[:, None] + np.arange(width) - width // 2
    c = np.where(c < 0, c + width, np.where(c >= n, c - width, c))  # whole rows at both ends
    c.sort(axis=1)
    v = np.where(c == np.arange(n)[:, None], 2.0 * width, -1.0)
    return np.arange(0, n * width + 1, width), c.reshape(-1), v.reshape(-1)


def test_copy_costs_a_few_updates():
    say("jacobi copy time")
    n = 400000
    rp, c, v = banded(n, 27)
    A = srtc.csr_from_host(rp, c, v, (n, n))
    b = torch.ones(n, dtype=torch.float64, device="cuda")
    ctx = srtc.Context(0)

    def solve():
        with pytest.raises(srtc.NotConverged):
            ctx.jacobi(A, b, torch.zeros_like(b), tol=0.0, max_iters=4)

    best = best_times(ctx, solve)
    # the copy moves A and itself, an update the copy and the vectors: 2.3 times
    # the bytes; one lane a row read A at a seventh of the rate
    assert best["jacobi.slice_copy"] <= 6 * best["jacobi.step"], best


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("width", [1, 2, 15, 16, 17, 31, 32, 33, 50])
def test_row_lengths(width, dtype):
    say("jacobi row length", width, dtype)
    n = 65536 + 70
    rp, c, v = banded(n, width)
    v = v.astype(oracle.NP_DTYPES[dtype])
    O = oracle.CSR(rp, c, v, n, n)
    A = srtc.csr_from_host(rp, c, v, (n, n))
    b = np.random.default_rng(width).uniform(-1, 1, n).astype(v.dtype)
    x = torch.zeros(n, dtype=torch.as_tensor(v).dtype, device="cuda")
    tol = 1e-9 if dtype == "f64" else 1e-3
    it, res = srtc.Context(0).jacobi(A, torch.as_tensor(b, device="cuda"), x, tol=tol)
    xo, lo, _, ok = oracle.jacobi(O, b, np.zeros(n, v.dtype), tol, dtype=dtype)
    assert ok and it == lo and res <= tol
    err = np.abs(x.cpu().numpy().astype(np.float64) - xo)
    assert np.all(err <= (1e-12 if dtype == "f64" else 1e-6) * (1 + np.abs(xo)))
