"""Parity cases derived from the library's own kernel planning.

`variant_cases()` finds, for every kernel instantiation compiled into
libo1d.so (o1d_kernel_variant), a small problem that the library's planner
(o1d_kernel_name, the same host code the entry points run) routes to it.  The
GPU parity suite runs every one of these cases against the oracle; the host
suite checks that no compiled variant is left without a case.  Only host-side
planning is called here: no GPU is needed to build the list.
"""
from __future__ import annotations

import functools

from paper_2309_15812_amd import _lib

OPS = {0: "fwd", 1: "bwd_input", 2: "bwd_weight", 3: "bwd"}


def _candidates():
    """Problem sizes (N, C, H, W, K, layout, aligned, stride, sampling), smallest first."""
    out = []
    # strip kernels: W a multiple of 4, aligned tensors, every tile stride
    for K in (7, 31, 33, 63):
        for M in range(4, 132, 4):
            for H, W in ((M, M), (max(1, M // 3), M), (max(1, M // 4), M), (M, max(4, (M // 3) // 4 * 4))):
                out.append((3, 4, H, W, K, _lib.O1D_NCHW, True, 1, _lib.O1D_FLOOR))
    # plane kernels: small NCHW planes with at least eight images
    for K in (7, 31, 63, 127):
        for H, W in ((14, 14), (16, 16), (5, 9), (13, 20), (40, 12), (40, 8)):
            out.append((8, 4, H, W, K, _lib.O1D_NCHW, True, 1, _lib.O1D_FLOOR))
            out.append((8, 4, H, W, K, _lib.O1D_NCHW, False, 1, _lib.O1D_FLOOR))
    # general kernels: ragged or unaligned NCHW, NHWC, small and large planes
    for K in (7, 31, 63, 127):
        for H, W in ((14, 14), (5, 9), (30, 30), (40, 33), (130, 70)):
            out.append((3, 4, H, W, K, _lib.O1D_NCHW, False, 1, _lib.O1D_FLOOR))
            out.append((3, 4, H, W, K, _lib.O1D_NHWC, True, 1, _lib.O1D_FLOOR))
    # walk kernels: calls of some size past the strip and plane kernels, every tile stride
    for K in (3, 15, 31, 47, 63):
        for H, W in ((14, 14), (13, 9), (27, 27), (30, 30), (38, 38), (47, 47), (49, 49), (57, 57), (56, 56), (61, 61),
                     (70, 26), (26, 70), (77, 77), (90, 16), (90, 42), (91, 91), (80, 27), (130, 130), (203, 203)):
            for size in (1.2e6, 2.4e6, 4.8e6):
                N = max(1, round(size / (64 * H * W)))
                out.append((N, 64, H, W, K, _lib.O1D_NHWC, True, 1, _lib.O1D_FLOOR))
                out.append((N, 64, H, W, K, _lib.O1D_NCHW, False, 1, _lib.O1D_FLOOR))
                out.append((N, 64, H, W, K, _lib.O1D_NCHW, True, 1, _lib.O1D_BILINEAR))
    out += [(10, 256, 36, 26, 5, _lib.O1D_NCHW, True, 1, _lib.O1D_BILINEAR),
            (7, 256, 25, 25, 27, _lib.O1D_NCHW, True, 1, _lib.O1D_BILINEAR),
            (51, 128, 18, 15, 1, _lib.O1D_NHWC, True, 1, _lib.O1D_FLOOR)]
    out.sort(key=lambda c: (c[0] * c[1] * c[2] * c[3] * c[4], c))
    return out


@functools.lru_cache(maxsize=None)
def variant_cases() -> dict:
    """{variant name: (N, C, H, W, K, dtype, layout, aligned, stride, sampling)} for every variant the planner reaches."""
    want = set(_lib.kernel_variants())
    found = {}
    for dt, dname in ((_lib.O1D_F32, "f32"), (_lib.O1D_BF16, "bf16")):
        for (N, C, H, W, K, layout, aligned, stride, sampling) in _candidates():
            plain = (layout, stride, sampling) == (_lib.O1D_NCHW, 1, _lib.O1D_FLOOR)
            for op in (0, 1, 2, 3) if plain else (0, 1, 2):
                name = _lib.kernel_name(op, N, C, H, W, K, stride, layout, sampling, dt, aligned)
                for v in name.split("+"):
                    if v in want and v not in found:
                        found[v] = (N, C, H, W, K, dname, "nhwc" if layout == _lib.O1D_NHWC else "nchw", aligned,
                                    stride, "bilinear" if sampling == _lib.O1D_BILINEAR else "floor")
            if len(found) == len(want):
                return found
    return found
