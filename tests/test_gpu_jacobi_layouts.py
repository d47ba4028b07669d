"""Jacobi steps on every layout of A (GPU): 64-row slices with 16-bit and
32-bit column offsets, rows too uneven for slices, systems too small for
them, row counts that no slice divides, runs that stop inside and at the end
of a replayed graph."""

import numpy as np
import pytest
import torch

import oracle
import paper_1512_00066_amd as srtc
from gpu_common import say

pytestmark = pytest.mark.gpu
TORCH = {"f64": torch.float64, "f32": torch.float32}


@pytest.fixture(scope="module")
def ctx():
    return srtc.Context(0)


def system(kind, n, dtype, seed):
    """(rows, cols, vals, b) of a diagonally dominant system."""
    rng = np.random.default_rng(seed)
    if kind == "banded":
        offs = np.array([-120, -7, -1, 1, 2, 90])
        r = np.repeat(np.arange(n), offs.size)
        c = r + np.tile(offs, n)
    elif kind == "edge16":  # the farthest offsets 16 bits hold
        offs = np.array([-32768, -3, 5, 32767])
        r = np.repeat(np.arange(n), offs.size)
        c = r + np.tile(offs, n)
    elif kind == "wide":
        r = np.repeat(np.arange(n), 6)
        c = rng.integers(0, n, r.size)
    else:  # uneven: one row in 50 long
        ln = np.where(np.arange(n) % 50 == 3, 90, 3)
        r = np.repeat(np.arange(n), ln)
        c = np.clip(r + rng.integers(-400, 400, r.size), 0, n - 1)
    keep = (c >= 0) & (c < n) & (c != r)
    k = np.unique(r[keep] * n + c[keep])
    r, c = k // n, k % n
    v = rng.uniform(-1, 1, r.size)
    dom = np.bincount(r, np.abs(v), n)
    d = (dom * 1.5 + 1) * np.where(rng.random(n) < 0.5, -1, 1)
    r, c, v = np.concatenate([r, np.arange(n)]), np.concatenate([c, np.arange(n)]), np.concatenate([v, d])
    dt = oracle.NP_DTYPES[dtype]
    return r, c, v.astype(dt), rng.uniform(-1, 1, n).astype(dt)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("kind,n", [("banded", 65536), ("banded", 65537), ("banded", 70001), ("edge16", 80000),
                                    ("wide", 66000), ("uneven", 70000), ("banded", 1), ("banded", 63),
                                    ("uneven", 5000)])
def test_layouts_match_oracle(ctx, kind, n, dtype):
    say("jacobi layout", kind, n, dtype)
    r, c, v, b = system(kind, n, dtype, 11)
    O = oracle.fold("plus_times", dtype, r, c, v, n, n)
    A = srtc.csr_from_host(O.rowptr, O.col, O.val, (n, n))
    bd = torch.as_tensor(b, device="cuda")
    tol = 1e-9 if dtype == "f64" else 1e-3
    xo, lo, ro, ok = oracle.jacobi(O, b, np.zeros(n, b.dtype), tol, dtype=dtype)
    assert ok
    # stops inside a run, at its end and one step into the next
    for k in {2, max(2, lo), lo + 1, lo + 2, 64}:
        x = torch.zeros(n, dtype=TORCH[dtype], device="cuda")
        it, res = ctx.jacobi(A, bd, x, tol=tol, steps_per_check=k)
        assert it == lo and res <= tol
        # rows sum at most 90 terms in fp64 and round once per update: fp64 a
        # few 2^-53 per update, fp32 2^-24, damped by the contraction
        err = np.abs(x.cpu().numpy().astype(np.float64) - xo)
        assert np.all(err <= (1e-12 if dtype == "f64" else 1e-6) * (1 + np.abs(xo)))


@pytest.mark.parametrize("n", [70001, 500])
def test_caps_and_nonfinite(ctx, n):
    say("jacobi caps", n)
    r, c, v, b = system("banded", n, "f64", 4)
    O = oracle.fold("plus_times", "f64", r, c, v, n, n)
    A = srtc.csr_from_host(O.rowptr, O.col, O.val, (n, n))
    bd = torch.as_tensor(b, device="cuda")
    for cap in (1, 2, 5, 8):
        x = torch.zeros(n, dtype=torch.float64, device="cuda")
        with pytest.raises(srtc.NotConverged):
            ctx.jacobi(A, bd, x, tol=0.0, max_iters=cap, steps_per_check=4)
        xo, lo, _, ok = oracle.jacobi(O, b, np.zeros(n), 0.0, max_iters=cap)
        assert not ok and lo == cap
        assert np.allclose(x.cpu().numpy(), xo, rtol=1e-12, atol=1e-15)
    # an infinite start: one update spreads it only to the rows that reach it
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    x[17] = float("inf")
    with pytest.raises(srtc.NotConverged):
        ctx.jacobi(A, bd, x, tol=0.0, max_iters=1, steps_per_check=2)
    reach = np.zeros(n, bool)
    for i in range(n) if n < 1000 else np.unique(np.clip(np.arange(17 - 130, 17 + 130), 0, n - 1)):
        reach[i] = 17 in O.col[O.rowptr[i]:O.rowptr[i + 1]] and i != 17
    assert np.array_equal(~np.isfinite(x.cpu().numpy()), reach)
