"""Contractions over rows that are no whole 16-byte items: the walk tap by tap, at its edges."""
import numpy as np
import pytest

from launches import launches
from paper_2201_05587_amd import api, harness
from paper_2201_05587_amd import workloads as wl


def record(cls, dtype, tm, tn, tk, wm, wn, stages, split_k=1, mfma=16):
    return api.make_schedule(cls, api.TT_SK_MFMA, tm, tn, tk, wm, wn, mfma, split_k, 1, 8 if dtype == wl.BF16 else 4, 8, stages)


def records(cls, dtype):
    k = 64 if dtype == wl.BF16 else 32
    return [record(cls, dtype, 32, 32, k, 16, 16, 2), record(cls, dtype, 64, 64, k // 2, 32, 32, 1, mfma=32 if dtype == wl.F32 else 16),
            record(cls, dtype, 64, 16, k // 2, 32, 16, 2), record(cls, dtype, 32, 32, k, 16, 16, 2, split_k=2), record(cls, dtype, 16, 64, k // 2, 16, 32, 2, split_k=3)]


def conv(dtype, n, c, h, w, k, f, stride, pad, cls=1):
    return wl.Kernel(cls, wl.ConvShape(n, c, h, w, k, f, f, stride, stride, pad, pad, dtype), 1, f"conv_{n}_{c}_{h}x{w}_{k}_{f}_s{stride}_p{pad}")


def product(dtype, batch, m, n, k):
    return wl.Kernel(7, wl.GemmShape(batch, m, n, k, 1, dtype), 1, f"product_{batch}_{m}_{n}_{k}")


# a pixel one element longer than items and one shorter, even and odd, one slice to many (an even and an odd number of them),
# filters larger than the image, no padding and more than the filter's half, strides, the tensor's last item, residuals;
# 17 and 21: too much padding, the walk along the run
CASES = [lambda d: conv(d, 1, 23, 5, 6, 33, 1, 1, 0), lambda d: conv(d, 2, 31, 7, 9, 40, 3, 1, 1), lambda d: conv(d, 1, 47, 6, 5, 66, 5, 1, 2),
         lambda d: conv(d, 3, 34, 11, 8, 17, 3, 2, 1), lambda d: conv(d, 1, 63, 3, 2, 64, 5, 1, 4), lambda d: conv(d, 1, 55, 8, 8, 31, 3, 1, 0),
         lambda d: conv(d, 2, 95, 4, 7, 48, 3, 1, 1, 2), lambda d: conv(d, 1, 17, 9, 9, 20, 3, 1, 1), lambda d: conv(d, 1, 21, 6, 7, 18, 5, 2, 2),
         lambda d: conv(d, 1, 130, 6, 6, 70, 3, 3, 1), lambda d: conv(d, 1, 257, 5, 5, 16, 1, 2, 0),
         lambda d: product(d, 3, 33, 70, 31), lambda d: product(d, 2, 65, 33, 63), lambda d: product(d, 1, 130, 17, 127), lambda d: product(d, 5, 18, 64, 201),
         lambda d: product(d, 1, 64, 66, 515)]
# of these every record applies: rows and columns for all of its tiles
CASES += [lambda d: conv(d, 2, 23, 9, 8, 66, 3, 1, 1), lambda d: conv(d, 3, 130, 17, 18, 70, 3, 3, 1), lambda d: conv(d, 2, 257, 12, 13, 66, 1, 2, 0),
          lambda d: conv(d, 1, 34, 17, 16, 65, 5, 2, 2), lambda d: conv(d, 2, 44, 9, 9, 66, 5, 1, 2), lambda d: conv(d, 1, 7 if d == wl.F32 else 55, 11, 7, 64, 3, 1, 1, 2),
          lambda d: product(d, 2, 66, 65, 127), lambda d: product(d, 1, 130, 70, 71)]


def by_taps(kernel):
    """The rule on the elements of a pixel (of a row): no whole items, more than one, and little padding."""
    s = kernel.shape
    item, c = (8 if s.dtype == wl.BF16 else 4), s.c if kernel.is_conv() else s.k
    padded = -(-c // item) * item
    if c % item == 0 or c <= item:
        return False
    return 7 * padded <= 8 * c if item == 4 else 5 * padded < 6 * c if c % 2 == 0 else 8 * padded <= 9 * c


def check_names(calls, walks):
    """Named as launched; `walks` says of a call whether it walks by taps (None: either)."""
    for (cls, shape, rec), want, (rc, made) in zip(calls, walks, launches(calls)):
        plan, which = api.tt_debug_launch(rec, cls, shape)
        assert rc == api.TT_OK and want in (None, which == api.TT_LAUNCH_TAPS), (shape, rec, made)
        assert made[0]["name"].startswith("tt::contract_taps_kernel<") == (which == api.TT_LAUNCH_TAPS)
        if plan.sketch == api.TT_SK_MFMA:
            assert made[0]["name"] == api.launched_name(rec, cls, shape)
            assert [made[0][x] for x in ("grid", "block", "lds")] == [plan.grid, plan.block, plan.lds_bytes]


def test_which_cases_walk_by_taps():
    """The cases above under their records, and channels to either side of the rule's lines."""
    calls, walks = [], []
    for dtype in (wl.F32, wl.BF16):
        lines = [conv(dtype, 8, c, 56, 56, 256, 3, 1, 1) for c in ((6, 7, 9, 13, 14, 15, 17) if dtype == wl.F32 else (10, 20, 22, 23, 35, 38, 43, 50, 63, 69))]
        for i, k in enumerate([make(dtype) for make in CASES] + lines):
            for rec in [None] + records(k.cls, dtype):
                if rec is None or api.tt_schedule_apply(rec, k.cls, k.shape).runnable():
                    calls.append((k.cls, k.shape, rec))
                    walks.append(None if rec is None else by_taps(k))
                else:
                    assert i < 16 or k in lines
    assert walks.count(True) > 120 and walks.count(False) > 40
    check_names(calls, walks)


def test_which_tiles_walk_by_taps():
    """Waves of at most 64 x 64, eight of them at most, and eight items a lane at most: every tile of the register pipeline."""
    calls, walks = [], []
    for v in range(api.lib.tt_num_variants()):
        dtype, family, tm, tn, tk, wm, wn, mf, bytes_, pipeline = api.tt_variant_info(v)[:10]
        if pipeline != 0 or family == 2 or bytes_ == 16:
            continue
        k = conv(dtype, 3, 511, 28, 28, 256, 3, 1, 1) if family == 0 else product(dtype, 1, 1300, 520, 511)
        rec = record(k.cls, dtype, tm, tn, tk, wm, wn, 1, mfma=mf)
        assert api.tt_schedule_apply(rec, k.cls, k.shape).variant_id == v
        waves = tm * tn // (wm * wn)
        calls.append((k.cls, k.shape, rec))
        walks.append(wm * wn <= 4096 and waves <= 8 and (tm + tn) * tk // (8 if dtype == wl.BF16 else 4) // (waves * 64) <= 8)
    assert walks.count(True) > 100 and walks.count(False) > 10
    check_names(calls, walks)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_walk_by_taps_against_the_oracle(case, dtype):
    import parity as P
    k = CASES[case](dtype)
    P.check_kernel(k, [None] + records(k.cls, dtype), seed=31 + case)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_what_lies_behind_a_pixel_is_not_read_into_it(dtype, bad):
    """The item that ends a pixel holds the next pixel's first elements, and a row's the next row's: of either operand."""
    import torch
    for k in (conv(dtype, 2, 23, 7, 9, 40, 1, 1, 0, 0), product(dtype, 2, 40, 36, 23)):
        inp = wl.make_inputs(k, 5)
        for rec in records(k.cls, dtype)[:2]:
            if not api.tt_schedule_apply(rec, k.cls, k.shape).runnable():
                continue
            dk = harness.device_kernel(k, 5, inp)
            a, b = (dk.tensors["a"], dk.tensors["b"]) if "a" in dk.tensors else (dk.tensors["x"], dk.tensors["w"])
            assert dk.run(rec) == api.TT_OK
            torch.cuda.synchronize()
            want = dk.output().clone().view(-1, dk.output().shape[-1])
            rows, columns = a.view(-1, 23), b.view(-1, 23)
            rows[1::2, 0] = bad      # of every second row, and of every third column
            columns[2::3, 0] = bad
            assert dk.run(rec) == api.TT_OK
            torch.cuda.synchronize()
            got = dk.output().view(-1, dk.output().shape[-1])
            n = got.shape[1]
            clean_rows = torch.arange(got.shape[0], device="cuda") % 2 == 0
            batch = columns.shape[0] // n
            for i in range(batch):  # (a product's batches have columns of their own)
                clean = torch.arange(i * n, (i + 1) * n, device="cuda") % 3 != 2
                part = slice(i * got.shape[0] // batch, (i + 1) * got.shape[0] // batch)
                keep = clean_rows[part][:, None] & clean[None, :]
                assert torch.equal(got[part][keep], want[part][keep]), (k.name, rec)
                assert not bool(torch.isfinite(got[part][~keep]).all())


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,c,f,tile,splits", [(wl.BF16, 34, 5, (32, 32, 32, 16, 16), 9), (wl.BF16, 44, 5, (32, 32, 32, 16, 16), 8), (wl.F32, 7, 5, (32, 32, 32, 16, 16), 4),
                                                   (wl.BF16, 63, 3, (64, 64, 32, 32, 32), 6), (wl.F32, 131, 1, (32, 32, 32, 16, 16), 5)])
def test_splits_share_the_walk(dtype, c, f, tile, splits):
    """A split adds up as many slices as any other, or one more: with ones for operands its partial sum counts the elements."""
    import torch
    k = conv(dtype, 1, c, 12, 12, 64, f, 2 if f == 1 else 1, f // 2)
    rec = record(k.cls, dtype, *tile, 2, split_k=splits)
    plan, which = api.tt_debug_launch(rec, k.cls, k.shape)
    assert which == api.TT_LAUNCH_TAPS
    splits, m, n = plan.eff_split_k, plan.M, plan.N
    dk = harness.device_kernel(k, 1)
    for t in ("x", "w"):
        dk.tensors[t].fill_(1.0)
    assert dk.run(rec) == api.TT_OK
    torch.cuda.synchronize()
    parts = dk.ws[:splits * m * n * 4].view(torch.float32).view(splits, m, n)
    inside = parts[:, k.shape.wo * (k.shape.ho // 2) + k.shape.wo // 2, :]  # (a pixel whose taps are all in the image)
    counts = inside[:, 0].tolist()
    assert bool((inside == inside[:, :1]).all()) and sum(counts) == c * f * f
    item, tk = (8 if dtype == wl.BF16 else 4), tile[2]
    slices = -(-f * f * -(-c // item) * item // tk)
    assert max(counts) <= -(-slices // splits) * tk, counts
    assert min(counts) > 0
