"""Convolutions over pixels that are not whole items, with the input rows of a tile in LDS."""
import numpy as np
import pytest

from paper_2201_05587_amd import api
from paper_2201_05587_amd import workloads as wl


def mfma(cls, tm, tn, split_k=1, order=0, vec=8):
    w = 32 if tm >= 32 and tn >= 32 else 16
    return api.make_schedule(cls, api.TT_SK_MFMA, tm, tn, 32, w, w, w, split_k, order, vec, 8, 2)


def conv(cls, n, c, h, w, k, r, s, stride, pad, dtype):
    return wl.Kernel(cls, wl.ConvShape(n, c, h, w, k, r, s, stride, stride, pad, pad, dtype), 1, f"c{c}_{h}x{w}_{r}x{s}_s{stride}_p{pad}")


# odd and even numbers of elements from pixel to pixel, tiles that end inside rows and images, images smaller than a tile,
# filters larger than the image, no padding and more than the filter's half, channels just short of an item
SHAPES = [(1, 3, 33, 32, 64, 7, 7, 2, 3), (3, 5, 15, 16, 40, 3, 3, 1, 1), (5, 1, 9, 16, 33, 7, 7, 1, 2), (4, 5, 14, 16, 96, 3, 3, 2, 0),
          (7, 6, 5, 8, 32, 3, 3, 1, 2), (2, 35, 20, 8, 70, 1, 1, 1, 0), (2, 11, 13, 8, 65, 3, 1, 1, 1), (1, 3, 64, 200, 64, 7, 7, 2, 3),
          (80, 5, 4, 8, 32, 3, 3, 3, 1), (1, 17, 19, 24, 48, 3, 3, 1, 1), (4, 3, 16, 40, 32, 7, 7, 4, 3), (1, 3, 17, 24, 130, 7, 7, 1, 3)]
TILES = [(128, 32), (256, 32), (128, 64), (256, 64), (128, 128)]
SMALL = [(32, 32), (64, 64)]  # the register pipeline


@pytest.mark.parametrize("shape", SHAPES)
def test_lds_holds_the_rows_of_every_tile(shape):
    """The launch's LDS against the filters and rows that the tiles need, counted tile by tile."""
    k = conv(1, *shape, wl.BF16)
    s, es, per_item = k.shape, 2, 8
    seen = 0
    for tm, tn in TILES:
        rec = mfma(1, tm, tn)
        if not api.tt_schedule_apply(rec, k.cls, s).runnable():
            continue
        plan, kernel = api.tt_debug_launch(rec, k.cls, s)
        if kernel != api.TT_LAUNCH_ROWS:
            continue
        seen += 1
        base = lambda m: (m // (s.ho * s.wo)) * (s.h + 2 * s.pad_h) + (m % (s.ho * s.wo)) // s.wo * s.stride_h
        rows = max(base(min(m + tm, plan.M) - 1) - base(m) + s.r for m in range(0, plan.M, tm))
        run = s.s * s.c
        last_word = ((s.wo - 1) * s.stride_w * s.c + -(-run // per_item) * per_item) * es + 4  # what a row's last pixel reads
        items = s.r * -(-run // per_item)
        assert plan.lds_bytes >= 2 * rows * last_word + tn * items * 16  # (the next tile's rows too)
        assert plan.lds_bytes <= 80 * 1024 and plan.block == (tm // 32) * (tn // (64 if tn % 64 == 0 and tm // 32 * (tn // 64) >= 4 else 32)) * 64
    assert seen or s.r * s.s == 1


@pytest.mark.parametrize("shape", [(32, 3, 224, 224, 64, 7, 7, 2, 3), (1, 3, 33, 32, 64, 7, 7, 2, 3), (4, 5, 14, 16, 96, 3, 3, 2, 0), (1, 3, 17, 24, 130, 7, 7, 1, 3)])
@pytest.mark.parametrize("count", [1, 3, 8])
def test_the_launch_has_the_workgroups_that_the_chip_holds(shape, count):
    """Whole columns of tiles, no more of them than there are tiles, and of all entries together no more than 256 CUs hold
    (but a column of each)."""
    k = conv(1, *shape, wl.BF16)
    for tm, tn in TILES:
        if not api.tt_schedule_apply(mfma(1, tm, tn), k.cls, k.shape).runnable():
            continue
        plan, kernel = api.tt_debug_launch(mfma(1, tm, tn), k.cls, k.shape, count)
        if kernel != api.TT_LAUNCH_ROWS:
            continue
        fit = min(160 * 1024 // plan.lds_bytes, 1024 // plan.block)
        columns, rows = -(-plan.N // tn), -(-plan.M // tm)
        assert plan.grid == columns * max(1, min(rows, 256 * fit // (columns * count)))


@pytest.mark.parametrize("shape", [
    # a row of 128 MB and more, whose layout in bytes is no number of 32 bits; padding as wide; images whose padded rows,
    # counted through all of them, are none
    (1, 1, 1, 1 << 26, 32, 17, 7, (1, 8), (16, 3)), (1, 1, 4, 1 << 27, 32, 7, 7, (1, 1), (3, 3)), (10, 1, 3, 8, 32, 17, 7, (1, 1 << 27), (8, 1 << 28)),
    (220000, 1, 1, 8, 32, 7, 7, (14, 1), (5000, 3))])
def test_sizes_that_no_layout_holds_keep_their_records(shape):
    n, c, h, w, k, r, s, stride, pad = shape
    cs = wl.ConvShape(n, c, h, w, k, r, s, *stride, *pad, wl.BF16)
    assert api.tt_debug_launch(mfma(1, 128, 32), 1, cs)[1] == api.TT_LAUNCH_RECORD


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [wl.F32, wl.BF16])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("cls", [wl.CLS_CONV2D_BIAS_RELU, wl.CLS_CONV2D_BIAS_ADD_RELU])
def test_rows_kernel(cls, shape, dt):
    import parity as P
    k = conv(cls, *shape, dt)
    recs = [mfma(cls, tm, tn, order=i % 6) for i, (tm, tn) in enumerate(TILES + SMALL)]
    recs = [r for r in recs if api.tt_schedule_apply(r, cls, k.shape).runnable()]
    ran = [api.tt_debug_launch(r, cls, k.shape)[1] for r in recs]
    assert bool(ran.count(api.TT_LAUNCH_ROWS)) == (dt == wl.BF16 and k.shape.r * k.shape.s > 1), ran
    P.check_kernel(k, [None] + recs, seed=31)


@pytest.mark.gpu
def test_infinities_reach_only_the_outputs_that_read_them():
    """Items carry elements of the next pixels and rows behind the run: those must not count, whatever they are."""
    import torch
    shape = api.to_c_shape(wl.ConvShape(2, 5, 12, 8, 32, 3, 3, 1, 1, 1, 1, wl.BF16))
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn((2, 12, 8, 5), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randn((32, 3, 3, 5), generator=g, device="cuda").to(x.dtype)
    bias = torch.zeros(32, device="cuda", dtype=x.dtype)
    rec = mfma(wl.CLS_CONV2D_ADD, 128, 32)
    assert api.tt_debug_launch(rec, wl.CLS_CONV2D_ADD, shape)[1] == api.TT_LAUNCH_ROWS
    run = lambda t: api.tt_conv2d_bias_relu(t, w, bias, None, shape, wl.CLS_CONV2D_ADD, rec).view(2, 12, 8, 32).float()
    clean = run(x)
    for img, p, q, value in ((0, 5, 4, float("inf")), (1, 11, 7, float("nan")), (0, 0, 0, float("-inf"))):
        bad = x.clone()
        bad[img, p, q, 3] = value
        got = run(bad)
        touched = torch.zeros((2, 12, 8), dtype=torch.bool, device="cuda")
        touched[img, max(p - 1, 0):p + 2, max(q - 1, 0):q + 2] = True
        assert torch.equal(got[~touched], clean[~touched])
        assert not torch.isfinite(got[touched]).any()
