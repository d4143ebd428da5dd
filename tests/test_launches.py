"""What the library asks the runtime for: kernels, grids and the LDS they are allowed."""
import pytest

from launches import launches
from paper_2201_05587_amd import api
from paper_2201_05587_amd import workloads as wl

ENABLED = 48 * 1024  # of dynamic LDS; more has to be asked for, per kernel


def mfma(cls, tm, tn, tk, wm, wn, mf, stages, vec, split_k=1, order=1):
    return api.make_schedule(cls, api.TT_SK_MFMA, tm, tn, tk, wm, wn, mf, split_k, order, vec, 8, stages)


def product(m, n, k, dtype):
    return wl.CLS_BATCH_MATMUL, wl.GemmShape(1, m, n, k, 1, dtype)


def test_lds_is_enabled_for_the_kernel_that_runs():
    """Two kernels under one record: rows of whole items, and not (either one first)."""
    calls = []
    for tile, first in (((128, 128, 64, 64, 64, 16), 0), ((128, 128, 64, 32, 64, 16), 1)):
        for k in ((6400, 6399), (6399, 6400))[first]:
            calls.append(product(8000, 8000, k, wl.BF16) + (mfma(wl.CLS_BATCH_MATMUL, *tile, 2, 8),))
    done = launches(calls)
    names = [made[0]["name"].split("<")[0] for rc, made in done]
    assert all(rc == api.TT_OK for rc, _ in done) and len(set(names)) == 2, names
    for rc, made in done:
        assert made[0]["lds"] > ENABLED and made[0]["enabled"] >= made[0]["lds"], done


def depthwise(n, c, h, w, stride, pad):
    return wl.CLS_DWCONV_BIAS_RELU6, wl.ConvShape(n, c, h, w, c, 3, 3, stride, stride, pad, pad, wl.F32)


def test_more_windows_than_are_counted():
    """Padding of many times the image: every record that applies runs, by the loop nest, in a grid that can be launched."""
    call = depthwise(1, 165, 4, 4, 1, 3700)  # nine thousand million outputs
    records = [None] + [api.make_schedule(wl.CLS_DWCONV_BIAS_RELU6, api.TT_SK_DWCONV, *r, 0, 1, 0, 1, 1, 1)
                        for r in ((8, 28, 32, 1, 7), (8, 28, 64, 2, 7), (8, 16, 16, 2, 2))]
    plans = [api.tt_schedule_apply(r, *call) for r in records if r is not None]
    assert all(p.runnable() for p in plans) and max(p.block for p in plans) == 1024
    for rec, (rc, made) in zip(records, launches([call + (r,) for r in records])):
        plan, _ = api.tt_debug_launch(rec, *call)
        assert rc == api.TT_OK and "dw_direct_kernel" in made[0]["name"], (rc, made)
        assert made[0]["grid"] * made[0]["block"] < 1 << 32
        assert (plan.sketch, plan.grid, plan.block) == (api.TT_SK_DIRECT, made[0]["grid"], made[0]["block"])


def test_output_rows_that_no_window_counts():
    """Rows of outputs beyond 2^31, over all images: a window would write at a negative row."""
    for n, c, pad, window in ((65536, 1, 16384, True), (65536, 1, 16385, False), (65536, 2, 16385, False)):
        call = wl.CLS_DWCONV_BIAS_RELU6, wl.ConvShape(n, c, 1, 1, c, 3, 3, 1, 1, pad, 1, wl.F32)
        assert (n * call[1].ho < 1 << 31) == window
        rec = api.make_schedule(wl.CLS_DWCONV_BIAS_RELU6, api.TT_SK_DWCONV, 8, 1, 32, 4, 1, 0, 1, 0, 1, 1, 1)
        (rc, made), = launches([call + (rec,)])
        assert rc == api.TT_OK and ("window" in made[0]["name"]) == window and ("dw_direct" in made[0]["name"]) != window


def test_rows_of_outputs_choose_the_instance():
    """Persistent kernels have an instance for rows that are whole 16-byte vectors and one for all others."""
    calls, odd = [], []
    for n in (64, 66, 72, 96, 100, 131):
        calls.append((1, wl.ConvShape(4, 3, 64, 64, n, 7, 7, 2, 2, 3, 3, wl.BF16), mfma(1, 128, 32, 32, 32, 32, 16, 2, 8)))
        calls.append((wl.CLS_DENSE_ADD, wl.GemmShape(1, 5000, n, 128, 1, wl.BF16), mfma(wl.CLS_DENSE_ADD, 64, 64, 64, 32, 32, 16, 7, 8)))
        calls.append((wl.CLS_DENSE_ADD, wl.GemmShape(1, 5000, n, 128, 1, wl.F32), mfma(wl.CLS_DENSE_ADD, 64, 64, 32, 32, 32, 16, 7, 4)))
        odd += [n % 8 != 0, n % 8 != 0, n % 4 != 0]
    for (cls, shape, rec), is_odd, (rc, made) in zip(calls, odd, launches(calls)):
        assert rc == api.TT_OK and made[0]["name"] == api.launched_name(rec, cls, shape)
        assert made[0]["name"].startswith(("tt::conv_rows_kernel<", "tt::gemm_stream_kernel<")) and made[0]["name"].endswith(f", {str(is_odd).lower()}>")


def test_tiles_of_one_item_a_lane_walk_by_taps_where_they_are_few():
    """Fp32 slices of 16 elements in four waves of 16 x 16: from 768 workgroups on, and long reductions, along the run."""
    def calls_of(tile, m, n, c, f, split=1, stages=2):
        cls, shape = (1, wl.ConvShape(1, c, m, 32, n, f, f, 1, 1, f // 2, f // 2, wl.F32)) if f else product(m * 32, n, c, wl.F32)
        return cls, shape, mfma(cls, *tile, 16, stages, 4, split)
    few, short = (32, 32, 16, 16, 16), (64, 16, 16, 16, 16)
    cases = [(calls_of(few, 64, 352, 57, 3), True), (calls_of(few, 64, 384, 57, 3), False), (calls_of(few, 64, 384, 55, 3), True), (calls_of(few, 64, 192, 131, 3, 2), False),
             (calls_of(few, 64, 192, 109, 3, 2), True), (calls_of(short, 128, 192, 57, 3), False), (calls_of(short, 128, 176, 57, 3), True), (calls_of(few, 64, 384, 131, 0), False),
             (calls_of(few, 64, 384, 127, 0), True), (calls_of((32, 32, 32, 16, 16), 64, 384, 57, 3), True), (calls_of((16, 16, 16, 16, 16), 64, 384, 57, 3), True)]
    for (call, taps), (rc, made) in zip(cases, launches([c for c, _ in cases])):
        assert rc == api.TT_OK and made[0]["name"].startswith("tt::contract_taps_kernel<" if taps else "tt::contract_kernel<"), (call, made)
        assert (api.tt_debug_launch(call[2], *call[:2])[1] == api.TT_LAUNCH_TAPS) == taps
