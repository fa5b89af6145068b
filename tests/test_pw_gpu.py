"""GPU parity of the block's matrix products at their edges: every combination of whole and cut runs of four
(pixels per image, channels, C'), k ranges that end inside a step and inside a 16-byte chunk, tiles that span images,
several pieces of the weight gradient's k.  Same bar as test_dsc_gpu.py."""
import pytest
import torch

import oracle
from paper_2309_15812_amd import ops
from test_dsc_gpu import DEV, TOL, dev, err, host, inputs

pytestmark = pytest.mark.gpu

CASES = [
    # N, C, C', H, W, dtype, offset in elements
    (3, 100, 36, 10, 10, "f32", 0),    # runs whole, k ends inside a step
    (3, 99, 35, 10, 10, "f32", 0),     # Wp's runs cut
    (3, 100, 36, 9, 11, "f32", 0),     # pixels' runs cut
    (5, 67, 131, 7, 9, "f32", 0),      # both
    (40, 160, 132, 6, 6, "f32", 0),    # many images per tile, several pieces of k
    (3, 100, 36, 10, 10, "f32", 2),    # unaligned tensors
    (3, 100, 132, 10, 10, "bf16", 0),
    (3, 99, 35, 10, 10, "bf16", 0),
    (3, 72, 36, 9, 11, "bf16", 0),
    (5, 67, 131, 7, 9, "bf16", 0),
    (40, 160, 132, 14, 14, "bf16", 0),
    (1, 1, 1, 1, 1, "f32", 0),
    (1, 8, 8, 2, 2, "f32", 0),         # pieces of k whose first step is cut
    (2, 8, 8, 18, 18, "f32", 0),
    (4, 8, 12, 18, 18, "bf16", 0),
    (3, 8, 17, 9, 11, "f32", 0),       # element loads of few channels: one, two and four columns per thread
    (3, 9, 16, 9, 11, "f32", 0),
    (4, 3, 140, 13, 13, "f32", 0),
    (3, 16, 33, 9, 11, "bf16", 0),
    (3, 17, 32, 9, 11, "bf16", 0),
    (4, 10, 10, 13, 13, "bf16", 0),
    (2, 32, 1, 7, 21, "bf16", 1),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_products(case):
    N, C, Co, H, W, dt, off = case
    d = inputs(N, C, Co, H, W, 3, dt, 90 + C)
    tdt = torch.float32 if dt == "f32" else torch.bfloat16
    x, dy = dev(d["x"], tdt, off), dev(d["dy_pw"], tdt, off)
    w, wp = dev(d["w"], tdt), dev(d["w_pw"], tdt, off)
    th = torch.from_numpy(d["theta"]).to(DEV)
    z, y = ops.dsc_fwd(x, w, th, wp)
    dx, dwd, dwp = ops.dsc_bwd(x, z, dy, w, th, wp)
    rz, ry = oracle.dsc_fwd(d["x"], d["w"], d["theta"], d["w_pw"])
    rdx, rdwd, rdwp = oracle.dsc_bwd(d["x"], d["dy_pw"], d["w"], d["theta"], d["w_pw"])
    for g, r in ((z, rz), (y, ry), (dx, rdx), (dwd, rdwd), (dwp, rdwp)):
        assert err(host(g), r) <= TOL[dt]


def test_k_past_the_end_is_not_multiplied():
    # infinite values in the last channel and pixel stay out of other rows (cleared, not multiplied by zero)
    N, C, Co, H, W = 2, 33, 20, 6, 6
    d = inputs(N, C, Co, H, W, 3, "f32", 5)
    x, w = dev(d["x"], torch.float32), dev(d["w"], torch.float32)
    wp = dev(d["w_pw"], torch.float32)
    wp[Co - 1, C - 1] = float("inf")
    th = torch.from_numpy(d["theta"]).to(DEV)
    z, y = ops.dsc_fwd(x, w, th, wp)
    _, ry = oracle.dsc_fwd(d["x"], d["w"], d["theta"], d["w_pw"])
    assert err(host(y)[:, :Co - 1], ry[:, :Co - 1]) <= 1e-5
    assert not torch.isfinite(y[:, Co - 1]).any()
