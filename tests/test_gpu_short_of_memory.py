"""Calls whose extra workspace the allocator refuses (GPU): they go on without
it, and their results meet the same bounds."""

import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_1512_00066_amd as srtc
from gen import synth
from gpu_common import say

pytestmark = pytest.mark.gpu


class Limited(srtc.Context):
    """A context whose allocator refuses requests of more than `limit` bytes."""

    def __init__(self, limit=None):
        super().__init__(0)
        srtc.lib().srtc_ctx_destroy(self._h)
        self._h = None
        self.limit, self.refused = limit, 0
        inner = self._cb

        def alloc(user, nbytes):
            if self.limit is not None and nbytes > self.limit:
                self.refused += 1
                return 0
            return inner[0](user, nbytes)

        self._cb = (srtc._ALLOC(alloc), inner[1])
        self._inner = inner
        h = ctypes.c_void_p()
        assert srtc.lib().srtc_ctx_create(0, self._cb[0], self._cb[1], None, ctypes.byref(h)) == 0
        self._h = h


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_dense_product_without_partial_sums(dtype):
    """64 x 64 x 5,000 splits k; without room for the parts it is one pass."""
    say("dense without workspace", dtype)
    g = torch.Generator().manual_seed(3)
    a, b = (torch.rand(s, generator=g, dtype=torch.float64).to(dtype) for s in ((64, 5000), (5000, 64)))
    exp = a.double() @ b.double()
    ctx = Limited()
    out = {}
    for limit in (None, 1 << 14):
        ctx.limit = limit
        C = torch.zeros((64, 64), dtype=dtype, device="cuda")
        ctx.contract("plus_times", "ik", a.cuda(), "kj", b.cuda(), "ij", C=C)
        out[limit] = C.cpu().double()
    assert ctx.refused > 0
    # positive terms: fp64 sums of 5,000 lose at most 5,000 2^-53; fp32 ones are
    # formed over at most 128 terms and joined in fp64, then rounded once
    tol = 5000 * 2.0**-53 if dtype == torch.float64 else 130 * 2.0**-24
    for got in out.values():
        assert torch.all((got - exp).abs() <= tol * exp)


def test_jacobi_without_the_copy_of_a():
    say("jacobi without the copy")
    n = 66000
    r = np.repeat(np.arange(n), 5)
    c = r + np.tile([-40, -1, 0, 1, 300], n)
    v = np.tile([-1.0, 0.5, 4.0, -0.25, 1.0], n)
    keep = (c >= 0) & (c < n)
    O = oracle.fold("plus_times", "f64", r[keep], c[keep], v[keep], n, n)
    A = srtc.csr_from_host(O.rowptr, O.col, O.val, (n, n))
    b = np.random.default_rng(1).uniform(-1, 1, n)
    xo, lo, _, ok = oracle.jacobi(O, b, np.zeros(n), 1e-9)
    assert ok
    ctx = Limited(int(1.5 * 8 * n))  # vectors only
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    it, res = ctx.jacobi(A, torch.as_tensor(b, device="cuda"), x, tol=1e-9)
    assert ctx.refused > 0 and it == lo and res <= 1e-9
    assert np.all(np.abs(x.cpu().numpy() - xo) <= 1e-12 * (1 + np.abs(xo)))


@pytest.mark.parametrize("n", [65, 130, 200])
def test_path_doubling_without_encoded_operands(n):
    """The 32-bit dense rounds from the path matrix itself."""
    say("apsp without words", n)
    src, dst, w = synth.dense_graph(n, 11, hi=50)
    w = w.astype(np.int32)
    O = oracle.fold("min_plus", "i32", dst, src, w, n, n)
    A = srtc.csr_from_host(O.rowptr, O.col, O.val, (n, n))
    Do, Ho, ro, _ = oracle.apsp_tiskin(O, inf_value=oracle.INT_INF)
    ld = (n + 63) // 64 * 64
    ctx = Limited()
    for limit in (None, 8 * ld * ld - 1):  # the words take 8 ld^2 bytes, P and its successor 8 n^2 each
        ctx.limit = limit
        D, H, rounds = ctx.apsp_tiskin(A)
        assert np.array_equal(D.cpu().numpy().astype(np.int64), Do)
        assert np.array_equal(H.cpu().numpy().astype(np.int64), Ho)
        assert rounds == ro
    assert ctx.refused == 1
