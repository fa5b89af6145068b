"""GPU parity of the walk kernels, at sizes that take them (the planner leaves small and narrow calls to the table
kernels); every test first checks by the planner's names that the operations it is about walk.

Same bar as test_parity_ex_gpu.py.  The cases cover planes as one tile and planes cut into regions, channel counts
that leave a partial block of four and channel runs without vector alignment, stacked small planes, every phase count,
both samplings, walks of one and of several chunks, and planes whose sides leave ragged strips.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_15812_amd import _lib, ops, synth
from test_parity_ex_gpu import DEV, err, run_ex, run_plain

pytestmark = pytest.mark.gpu

FWD, DX, DW, BOTH = 0, 1, 2, 3  # y, dx, dw, and dx and dw in one pass


def assert_walks(walks, N, C, H, W, K, dtype, stride=1, layout="nchw", sampling="floor", aligned=True):
    for op in walks:
        name = _lib.kernel_name(op, N, C, H, W, K, stride, int(layout == "nhwc"), int(sampling == "bilinear"),
                                int(dtype == "bf16"), aligned)
        assert name.startswith("walk_"), (op, name)


EX = [
    # N, C, H, W, K, dtype, theta, stride, layout, sampling, offset in elements, operations that walk
    (64, 128, 14, 14, 7, "f32", "zero", 1, "nhwc", "floor", 0, (DW,)),         # small planes, stacked
    (60, 97, 13, 9, 31, "f32", "uniform", 1, "nhwc", "floor", 0, (0, 1, 2)),   # small, ragged, a block of one channel
    (33, 98, 14, 14, 31, "bf16", "uniform", 1, "nhwc", "bilinear", 0, (0, 1, 2)),
    (43, 88, 9, 5, 47, "bf16", "uniform", 1, "nhwc", "floor", 1, (0, 1, 2)),   # small, no vector alignment
    (70, 90, 7, 3, 63, "f32", "uniform", 1, "nhwc", "floor", 0, (0, 1, 2)),    # line longer than the plane
    (12, 58, 56, 56, 31, "f32", "discrete8", 1, "nhwc", "floor", 0, (0, 1, 2)),  # one tile per channel
    (4, 21, 138, 130, 15, "f32", "uniform", 1, "nhwc", "floor", 0, (0, 1, 2)),   # regions
    (2, 41, 117, 132, 31, "bf16", "uniform", 1, "nhwc", "floor", 0, (0, 1, 2)),  # odd channel count: element accesses
    (2, 42, 117, 132, 31, "bf16", "uniform", 1, "nhwc", "floor", 1, (0, 1, 2)),  # the same by the address
    (8, 57, 50, 56, 15, "bf16", "uniform", 1, "nhwc", "bilinear", 0, (0, 1, 2)),
    (18, 30, 40, 40, 47, "f32", "uniform", 1, "nhwc", "floor", 0, (0, 1, 2)),
    (6, 60, 100, 60, 63, "f32", "uniform", 2, "nhwc", "floor", 0, (0, 1, 2)),    # four phases
    (27, 27, 45, 63, 47, "bf16", "uniform", 2, "nhwc", "floor", 0, (0, 1, 2)),   # odd channel count
    (12, 50, 100, 91, 31, "f32", "uniform", 3, "nhwc", "bilinear", 0, (0, 1, 2)),  # nine phases, uneven last ones
    (11, 33, 169, 129, 15, "f32", "uniform", 2, "nchw", "floor", 0, (FWD, DW)),
    (5, 78, 131, 155, 15, "bf16", "uniform", 2, "nchw", "bilinear", 0, (FWD, DW)),
    (5, 62, 248, 232, 15, "f32", "uniform", 3, "nchw", "floor", 0, (FWD, DW)),
    (12, 60, 56, 56, 31, "f32", "uniform", 1, "nchw", "bilinear", 0, (0, 1, 2)),
    (6, 64, 63, 117, 63, "bf16", "uniform", 1, "nchw", "bilinear", 0, (0, 1, 2)),
]
PLAIN = [
    # N, C, H, W, K, dtype, offset in elements, operations that walk
    (5, 130, 56, 56, 63, "f32", 0, (DW, BOTH)),        # sums of more than 32 cells
    (9, 23, 116, 111, 15, "f32", 0, (0, 1, 2, 3)),     # odd width
    (2, 105, 113, 107, 15, "bf16", 0, (0, 1, 2, 3)),
    (1, 65, 218, 162, 15, "bf16", 0, (0, 1, 2, 3)),    # regions
    (6, 20, 199, 199, 51, "f32", 0, (0, 1, 2, 3)),
    (32, 80, 45, 37, 15, "bf16", 0, (BOTH,)),
    (20, 70, 56, 54, 3, "bf16", 1, (DW, BOTH)),        # tensors without vector alignment
    (22, 60, 56, 56, 1, "f32", 1, (DW, BOTH)),
]


@pytest.mark.parametrize("case", EX, ids=lambda c: "-".join(map(str, c[:11])))
def test_walk_ex(case):
    N, C, H, W, K, dtype, theta, s, layout, sampling, offset, walks = case
    assert_walks(walks, N, C, H, W, K, dtype, s, layout, sampling, aligned=offset == 0)
    run_ex(N, C, H, W, K, dtype, theta, s, layout, sampling, offset=offset, label=f"walk {case}")


@pytest.mark.parametrize("case", PLAIN, ids=lambda c: "-".join(map(str, c[:7])))
def test_walk_plain(case):
    N, C, H, W, K, dtype, offset, walks = case
    assert_walks(walks, N, C, H, W, K, dtype, aligned=offset == 0)
    run_plain(N, C, H, W, K, dtype, offset=offset, label=f"walk {case}")


def test_walk_keeps_channels_apart():
    # an infinite pixel and a non-finite angle stay in their channels (four channels share a workgroup)
    N, C, H, W, K = 20, 40, 56, 57, 47
    assert_walks((0, 1, 2), N, C, H, W, K, "f32", 1, "nhwc")
    d = synth.make_inputs(synth.Workload("apart", N, C, H, W, K, "f32", "uniform", "fwd+bwd", 7))
    d["theta"][5] = np.nan
    x = torch.from_numpy(np.ascontiguousarray(d["x"].transpose(0, 2, 3, 1))).to(DEV)
    dy = torch.from_numpy(np.ascontiguousarray(d["dy"].transpose(0, 2, 3, 1))).to(DEV)
    x[0, :, :, 0] = float("inf")
    dy[1, H - 1, :, 2] = float("-inf")
    w, th = torch.from_numpy(d["w"]).to(DEV), torch.from_numpy(d["theta"]).to(DEV)
    y = ops.fwd_ex(x, w, th, 1, "nhwc").cpu().numpy()
    dx = ops.bwd_input_ex(dy, w, th, (H, W), 1, "nhwc").cpu().numpy()
    dw = ops.bwd_weight_ex(x, dy, th, K, 1, "nhwc").cpu().numpy()
    assert np.isnan(y[..., 5]).all() and np.isnan(dx[..., 5]).all() and np.isnan(dw[5]).all()
    keep = [c for c in range(C) if c not in (0, 2, 5)]
    args = d["w"][keep], d["theta"][keep]
    assert err(y[..., keep].transpose(0, 3, 1, 2), oracle.fwd(d["x"][:, keep], *args)) <= 1e-5
    assert err(dx[..., keep].transpose(0, 3, 1, 2), oracle.bwd_input(d["dy"][:, keep], *args)) <= 1e-5
    assert err(dw[keep], oracle.bwd_weight(d["x"][:, keep], d["dy"][:, keep], d["theta"][keep], K)) <= 1e-5


def test_walk_weight_gradient_is_reproducible():
    N, C, H, W, K = 6, 96, 56, 56, 31
    assert_walks((DW,), N, C, H, W, K, "f32", 1, "nhwc", "bilinear")
    x = torch.randn(N, H, W, C, device=DEV)
    dy = torch.randn(N, H, W, C, device=DEV)
    th = torch.rand(C, device=DEV) * 180
    a = ops.bwd_weight_ex(x, dy, th, K, 1, "nhwc", "bilinear")
    assert torch.equal(a, ops.bwd_weight_ex(x, dy, th, K, 1, "nhwc", "bilinear"))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("layout,sampling", [("nhwc", "floor"), ("nhwc", "bilinear"), ("nchw", "floor")])
@pytest.mark.parametrize("stride", [1, 2, 3])
def test_non_finite_angles_poison_their_channels(stride, layout, sampling, dtype):
    # y and dx of such a channel are NaN at every pixel, also where no tap of any finite angle would land (stride
    # phases without cells), dw at every tap; the other channels (four share an NHWC workgroup) stay finite.
    N, C, H, W, K = 48, 64, 80, 80, 47
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    if layout == "nhwc":
        assert_walks((0, 1, 2), N, C, H, W, K, dtype, stride, layout, sampling)
    P, Q = ops.out_size(H, stride), ops.out_size(W, stride)
    rand = torch.Generator(device=DEV).manual_seed(3)

    def plane(h, w):
        return torch.randn((N, h, w, C) if layout == "nhwc" else (N, C, h, w), generator=rand, device=DEV).to(dt)

    x, dy = plane(H, W), plane(P, Q)
    w = torch.randn(C, K, generator=rand, device=DEV).to(dt)
    th = torch.rand(C, generator=rand, device=DEV) * 180
    bad = [1, 2, 7, C - 1]
    th[bad] = torch.tensor([float("nan"), float("inf"), float("-inf"), float("nan")], device=DEV)
    how = (stride, layout, sampling)
    y, dx = ops.fwd_ex(x, w, th, *how), ops.bwd_input_ex(dy, w, th, (H, W), *how)
    dw = ops.bwd_weight_ex(x, dy, th, K, *how)
    good = [c for c in range(C) if c not in bad]
    for t in (y, dx, dw):
        t = t.movedim(-1, 1) if layout == "nhwc" and t.dim() == 4 else t
        t = t.movedim(1, 0) if t.dim() == 4 else t
        assert torch.isnan(t[bad]).all() and torch.isfinite(t[good]).all()


NONFINITE = [
    # N, C, H, W, K, dtype, stride, layout, sampling
    (8, 64, 57, 57, 31, "f32", 1, "nhwc", "floor"),       # 57 rows: two strips of 28 reach 27 rows past the plane
    (8, 64, 57, 57, 31, "bf16", 1, "nhwc", "bilinear"),
    (64, 70, 13, 14, 31, "f32", 1, "nhwc", "floor"),      # small planes, idle lanes
    (40, 64, 57, 57, 47, "f32", 2, "nhwc", "floor"),
    (4, 64, 57, 57, 31, "f32", 1, "nchw", "bilinear"),
    (11, 33, 169, 129, 15, "f32", 2, "nchw", "floor"),    # regions that end past the plane
    (2, 105, 113, 107, 15, "bf16", 1, "nchw", "floor"),   # also both gradients in one pass
    (5, 130, 56, 56, 63, "f32", 1, "nchw", "floor"),
]


@pytest.mark.parametrize("case", NONFINITE, ids=lambda c: "-".join(map(str, c)))
def test_weight_gradients_keep_non_finite_pixels_to_their_taps(case):
    # an infinite or NaN pixel reaches the taps that read it and no other: same finite taps, infinities and NaN as the
    # oracle, same values (float32: 1e-5 of the largest finite one, bfloat16: 2e-2)
    N, C, H, W, K, dtype, s, layout, sampling = case
    plain = (s, layout, sampling) == (1, "nchw", "floor")
    assert_walks((DW, BOTH) if plain else (DW,), N, C, H, W, K, dtype, s, layout, sampling)
    d = synth.make_inputs(synth.Workload("nonfinite", N, C, H, W, K, dtype, "uniform", "fwd+bwd", 11))
    d["theta"][:4] = [0, 45, 112.5, 90]
    P, Q = oracle.out_size(H, s), oracle.out_size(W, s)
    x, dy = d["x"], d["dy"][:, :, :P, :Q].copy()
    ys, xs = s * ((P - 1) // 2), s * ((Q - 1) // 2)
    spots = [(0, 0), (0, s * (Q - 1)), (s * (P - 1), 0), (s * (P - 1), s * (Q - 1)), (ys, xs)]

    def spoil(t, step):
        for c, v in ((0, np.inf), (1, -np.inf), (2, np.nan), (3, np.inf), (C - 1, np.inf)):
            p, q = spots[(c + (c == C - 1)) % 5]
            t[c % N, c, p // step, q // step] = v

    tdtype = torch.float32 if dtype == "f32" else torch.bfloat16

    def put(t):
        t = t.transpose(0, 2, 3, 1) if layout == "nhwc" else t
        return torch.from_numpy(np.ascontiguousarray(t)).to(DEV).to(tdtype)

    def same(g, r):
        g = g.float().cpu().numpy()
        assert (np.isnan(g) == np.isnan(r)).all() and (np.isposinf(g) == np.isposinf(r)).all()
        assert (np.isneginf(g) == np.isneginf(r)).all()
        fin = np.isfinite(r)
        assert fin[:4].any() and not fin[:4].all() and fin[4:C - 1].all()
        assert err(g[fin], r[fin]) <= (1e-5 if dtype == "f32" else 2e-2)

    th = torch.from_numpy(d["theta"]).to(DEV)
    clean = x.copy()
    spoil(x, 1)
    same(ops.bwd_weight_ex(put(x), put(dy), th, K, s, layout, sampling),
         oracle.bwd_weight(x, dy, d["theta"], K, stride=s, mode=sampling))
    if plain:
        # the one-pass backward holds x in registers and walks dy
        spoil(dy, s)
        _, dw = ops.bwd(put(clean), put(dy), torch.from_numpy(d["w"]).to(DEV).to(tdtype), th)
        same(dw, oracle.bwd_weight(clean, dy, d["theta"], K))
