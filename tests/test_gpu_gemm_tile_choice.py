"""Which tile a dense product takes (GPU): rows that a tile of 128 would pad
cost what they are, not what it covers."""

import pytest
import torch

import paper_1512_00066_amd as srtc
from gpu_common import say
from gpu_profile import best_times

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_padded_rows_are_not_multiplied(dtype):
    """192 rows are three tiles of 64, 256 rows two of 128: three quarters of
    the work, at whichever rate the tiles reach."""
    say("gemm tile choice", dtype)
    ctx = srtc.Context(0)
    ms = {}
    for m in (192, 256):
        A, B = torch.rand(m, 2000, device="cuda", dtype=dtype), torch.rand(2000, 16384, device="cuda", dtype=dtype)
        C = torch.empty(m, 16384, device="cuda", dtype=dtype)
        call = lambda: ctx.contract("plus_times", "ik", A, "kj", B, "ij", C=C)
        call()
        ms[m] = sum(best_times(ctx, call, 10).values())
    assert ms[192] <= 0.92 * ms[256], ms
