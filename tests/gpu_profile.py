"""Times of a call's profiled kernels, from the library's own events."""

import ctypes

import paper_1512_00066_amd as srtc


def best_times(ctx, call, runs=6):
    """{profile entry: least milliseconds a launch} over some runs of `call`."""
    L, best = srtc.lib(), {}
    name, n, ms, by = ctypes.create_string_buffer(96), ctypes.c_int64(), ctypes.c_double(), ctypes.c_double()
    for _ in range(runs):
        L.srtc_profile_enable(ctx._h, 1)
        try:
            call()
            i = 0
            while L.srtc_profile_query(ctx._h, i, name, 96, ctypes.byref(n), ctypes.byref(ms), ctypes.byref(by)) == 0:
                key = name.value.decode()
                best[key] = min(best.get(key, float("inf")), ms.value / n.value)
                i += 1
        finally:
            L.srtc_profile_enable(ctx._h, 0)
    return best
