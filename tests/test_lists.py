"""Lists of kernels: which entries share a launch (host), and that shared launches compute every entry (GPU)."""
import ctypes
import random

import numpy as np
import pytest

from paper_2201_05587_amd import api
from paper_2201_05587_amd import workloads as wl


def mfma(cls, tm, tn, tk, wm, wn, mf, split_k=1, order=0, vec=8, unroll=8, stages=3):
    return api.make_schedule(cls, api.TT_SK_MFMA, tm, tn, tk, wm, wn, mf, split_k, order, vec, unroll, stages)


# ---- on the host: addresses are made up, nothing is launched -------------------------------------------------------
class FakeList(api.KernelList):
    def __init__(self, entries):
        """entries: (kernel, record, [addresses of x, w, bias, res, y], workspace address)"""
        self.keep, self.scheds = [], []
        self.n = len(entries)
        self.descs = (api.tt_kernel_desc * max(self.n, 1))()
        self.ptrs = (ctypes.POINTER(api.tt_schedule) * max(self.n, 1))()
        for i, (kernel, rec, at, ws) in enumerate(entries):
            d, shape = self.descs[i], api.to_c_shape(kernel.shape)
            self.keep.append(shape)
            d.cls, d.use_count, d.shape = kernel.cls, kernel.use_count, ctypes.addressof(shape)
            slots = (0, 1, 2, 3, 4) if kernel.cls in api.CONV_CLASSES else (0, 1, 4) if kernel.cls == api.TT_BATCH_MATMUL else (0, 1, 2, 4)
            for slot, which in enumerate(slots):
                d.bufs[slot] = at[which] or None
            d.ws, d.ws_bytes = ws, (1 << 30) if ws else 0
            if rec is not None:
                self.scheds.append(rec)
                self.ptrs[i] = ctypes.pointer(rec)


def ranges(kernel, at, ws, ws_bytes):
    """(ranges written, ranges read) of an entry."""
    s = kernel.shape
    es = 2 if s.dtype == wl.BF16 else 4
    if kernel.cls in api.CONV_CLASSES or kernel.cls == api.TT_DWCONV_BIAS_RELU6:
        filters = s.k * s.r * s.s * (1 if kernel.cls == api.TT_DWCONV_BIAS_RELU6 else s.c)
        sizes = (s.n * s.h * s.w * s.c, filters, s.k, s.n * s.ho * s.wo * s.k, s.n * s.ho * s.wo * s.k)
    else:
        sizes = (s.batch * s.m * s.k, s.batch * s.n * s.k, s.n, 0, s.batch * s.m * s.n)
    spans = [(a, a + z * es) for a, z in zip(at, sizes)]
    used = [spans[i] for i in range(4) if at[i]]
    return [spans[4]] + ([(ws, ws + ws_bytes)] if ws_bytes else []), used


def test_windows_keep_dependent_entries_in_order():
    """Random lists over a few overlapping tensors: an entry that touches what an earlier one writes, or writes what an
    earlier one touches, is launched behind it; every entry is launched once, and launches hold one data type and
    family, or one plan."""
    conv = lambda c, k, hw, f, dt, cls=1: wl.Kernel(cls, wl.ConvShape(1, c, hw, hw, k, f, f, 1, 1, f // 2, f // 2, dt))
    shapes = [conv(64, 64, 14, 3, wl.BF16), conv(64, 64, 14, 1, wl.BF16), conv(32, 64, 14, 3, wl.BF16, 2), conv(64, 64, 14, 3, wl.F32),
              wl.Kernel(4, wl.GemmShape(1, 196, 64, 64, 1, wl.BF16)), wl.Kernel(7, wl.GemmShape(4, 49, 64, 64, 1, wl.BF16)),
              wl.Kernel(7, wl.GemmShape(4, 49, 64, 64, 0, wl.BF16)), wl.Kernel(4, wl.GemmShape(1, 1, 64, 64, 1, wl.F32)),
              wl.Kernel(8, wl.ConvShape(1, 64, 14, 14, 64, 3, 3, 1, 1, 1, 1, wl.F32)), conv(3, 64, 28, 7, wl.BF16)]
    rng = random.Random(11)
    shared, followed = 0, 0
    for _ in range(200):
        entries, spans = [], []
        for _ in range(rng.randint(2, 40)):
            k = rng.choice(shapes)
            at = [(1 << 20) * rng.randint(1, 60) + 16 * rng.randint(0, 4000) for _ in range(5)]
            if k.cls != 2:
                at[3] = 0
            if k.cls == api.TT_BATCH_MATMUL:
                at[2] = 0
            rec, ws, ws_bytes = None, 0, 0
            if k.cls in (1, 2, 4) and rng.random() < 0.3 and k.shape.dtype == wl.F32:
                rec = mfma(k.cls, 32, 32, 32, 16, 16, 16, split_k=2, vec=4)
                plan = api.tt_schedule_apply(rec, k.cls, k.shape)
                if plan.status != api.TT_OK:
                    rec = None
                else:
                    ws, ws_bytes = (1 << 20) * rng.randint(1, 60), plan.workspace_bytes
            entries.append((k, rec, at, ws))
            spans.append(ranges(k, at, ws, ws_bytes))
        listed = FakeList(entries).launches()
        overlap = lambda xs, ys: any(a < d and c < b for a, b in xs for c, d in ys)
        for j in range(len(entries)):
            assert listed[j].launch >= 0
            for i in range(j):
                (wi, ri), (wj, rj) = spans[i], spans[j]
                if overlap(wi, wj) or overlap(wi, rj) or overlap(ri, wj):
                    assert listed[i].launch < listed[j].launch, (i, j)
                    followed += 1
        by_launch = {}
        for (k, rec, _, _), l in zip(entries, listed):
            by_launch.setdefault(l.launch, []).append((k, rec, l))
        assert sorted(by_launch) == list(range(len(by_launch)))
        for members in by_launch.values():
            assert all(l.entries == len(members) for _, _, l in members) and len(members) <= 20
            assert len({k.shape.dtype for k, _, _ in members}) == 1
            assert len({(l.listed, l.tile_m, l.tile_n) for _, _, l in members}) == 1
            if not members[0][2].listed:
                assert len({(k.cls, k.shape, rec is None) for k, rec, _ in members}) == 1 and len(members) <= 8
            shared += len(members) > 1
    assert shared > 100 and followed > 1000


def test_entries_that_run_several_times_or_not_at_all():
    k = wl.Kernel(4, wl.GemmShape(1, 196, 64, 64, 1, wl.BF16))
    at = lambda i: [(1 << 24) * (5 * i + j + 1) for j in range(5)]
    fake = FakeList([(k, None, at(i), 0) for i in range(5)])
    assert [l.launch for l in fake.launches()] == [0] * 5
    fake.descs[1].use_count = 0
    fake.descs[3].use_count = 2  # runs by itself, between the windows around it
    assert [l.launch for l in fake.launches()] == [0, -1, 0, 1, 2]
    fake.descs[4].bufs[0] = None
    with pytest.raises(api.TTError):
        fake.launches()


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F32])
@pytest.mark.parametrize("m, k", [(1 << 20, 256), (1 << 19, 512)])
def test_shared_launches_stay_below_the_largest_grid(dtype, m, k):
    """A launch holds less than 2^32 threads, and a workgroup here at most 1024."""
    kernel = wl.Kernel(4, wl.GemmShape(1, m, 768, k, 1, dtype))
    other = wl.Kernel(4, wl.GemmShape(1, m + 1, 768, k, 1, dtype))
    at = lambda i: [(1 << 34) * (5 * i + j + 1) for j in range(5)]
    entries = [((kernel, other)[i % 2], None, at(i), 0) for i in range(40)]
    listed = FakeList(entries).launches()
    for launch in {l.launch for l in listed if l.listed}:
        members = [(e[0].shape, l) for e, l in zip(entries, listed) if l.launch == launch]
        grid = sum(-(-s.m // l.tile_m) * -(-s.n // l.tile_n) for s, l in members)
        assert len(members) == 1 or grid <= 1 << 21, (len(members), grid)


@pytest.mark.parametrize("stride", [1, 2])
def test_shared_depthwise_launches_stay_below_the_largest_grid(stride):
    """Maps of one pixel just below the 2 GiB that a shared launch reads: four channels a thread, and all can read one input."""
    n, c = (1 << 15) - 1, 1 << 14
    kernel = wl.Kernel(8, wl.ConvShape(n, c, 1, 1, c, 3, 3, stride, stride, 1, 1))
    at = lambda i: [1 << 34, 1 << 33, 0, 0, (1 << 34) * (i + 2)]
    listed = FakeList([(kernel, None, at(i), 0) for i in range(36)]).launches()
    assert all(l.listed for l in listed)
    for launch in {l.launch for l in listed}:
        members = sum(l.launch == launch for l in listed)
        assert members * -(-n * (c // 4) // 256) <= 1 << 21, members


def test_shared_launches_of_streams_stay_below_the_largest_grid():
    """Reductions of 16, 16 columns, as many rows as the loads' offsets hold: a workgroup has at most 512 of them."""
    kernel = wl.Kernel(4, wl.GemmShape(1, (1 << 25) - 1, 16, 16, 1, wl.F32))
    rec = mfma(4, 32, 16, 16, 32, 16, 16, vec=4)
    at = lambda i: [1 << 34, 1 << 33, 0, 0, (1 << 34) * (i + 2)]
    listed = FakeList([(kernel, rec, at(i), 0) for i in range(48)]).launches()
    assert all(l.listed for l in listed)
    for launch in {l.launch for l in listed}:
        assert sum(l.launch == launch for l in listed) * ((1 << 25) // 512) <= 1 << 21


def list_ends():
    ring = lambda m, n, k, tile: (wl.Kernel(4, wl.GemmShape(1, m, n, k, 1, wl.BF16)), mfma(4, *tile))
    conv = (wl.Kernel(1, wl.ConvShape(1, 128, 28, 28, 128, 3, 3, 1, 1, 1, 1, wl.BF16)), mfma(1, 64, 64, 64, 32, 32, 16))
    stream = lambda m, n, k: (wl.Kernel(4, wl.GemmShape(1, m, n, k, 1, wl.F32)), mfma(4, 32, 32, 32, 16, 16, 16, vec=4))
    dw = (wl.Kernel(8, wl.ConvShape(2, 32, 28, 28, 32, 3, 3, 1, 1, 1, 1)), None)
    return {
        # name -> (entries, sizes of their launches); a launch of one is a choice only where its record names the tile
        "apart": ([ring(4096, 4096, 4096, (128, 256, 64, 32, 64, 16)), ring(64, 64, 64, (32, 32, 64, 16, 16, 16))], [1, 1]),
        "together": ([ring(4096, 4096, 4096, (64, 64, 32, 32, 32, 16)), ring(64, 64, 64, (32, 32, 32, 16, 16, 16))], [2]),
        # one more than a launch takes: of contractions, streams, depthwise entries
        "tail": ([conv] * 21, [2, 19]), "streams": ([stream(9000, 64, 32)] * 49, [2, 47]), "depthwise": ([dw] * 37, [2, 35]),
        # nothing to share with
        "one": ([conv], [1]), "one_stream": ([stream(9000, 64, 32)], [1]), "one_depthwise": ([dw], [1]),
        "beside_streams": ([stream(9000, 64, 32)] * 2 + [stream(64, 64, 640)], [1, 2]),
        "two_families": ([conv, ring(64, 64, 64, (32, 32, 64, 16, 16, 16))], [1, 1]),
    }


@pytest.mark.parametrize("name", list(list_ends()))
def test_an_entry_that_shares_no_launch_keeps_its_record(name):
    entries, sizes = list_ends()[name]
    at = lambda i: [(1 << 34) * (5 * i + j + 1) if j != 3 else 0 for j in range(5)]
    listed = FakeList([(k, rec, at(i), 0) for i, (k, rec) in enumerate(entries)]).launches()
    assert sorted(l.entries for l in {l.launch: l for l in listed}.values()) == sizes
    for (k, rec), l in zip(entries, listed):
        assert bool(l.listed) == (l.entries > 1)
        if l.entries == 1:
            plan = api.tt_debug_launch(rec, k.cls, k.shape)[0]
            assert (l.tile_m, l.tile_n, l.tile_k) == (plan.tile_m, plan.tile_n, plan.tile_k)


def test_launches_name_the_kernel_and_the_tile_they_run_in():
    """Whatever tiles the records name: depthwise windows of 4 x 2 and, at stride two, 2 x 2 outputs of four channels, streams in
    blocks of 16 x 16 on the shortest instance that holds the reduction, contractions in a tile of the rule."""
    dw = lambda stride: (wl.Kernel(8, wl.ConvShape(1, 32, 13, 13, 32, 3, 3, stride, stride, 1, 1)),
                         api.make_schedule(8, api.TT_SK_DWCONV, 4, 4, 8, 1, 2, 0, 1, 0, 4, 1, 1))
    stream = lambda k, n: (wl.Kernel(4, wl.GemmShape(1, 90000, n, k, 1, wl.F32)), mfma(4, 32, 32, 16, 16, 16, 16, vec=4))
    tiles = (wl.Kernel(5, wl.GemmShape(1, 300, 1032, 96, 1, wl.BF16)), mfma(5, 128, 256, 64, 32, 64, 16))
    lone = (wl.Kernel(7, wl.GemmShape(3, 50, 64, 50, 0, wl.BF16)), None)
    entries = [dw(1), dw(2), stream(32, 64), stream(20, 64), stream(36, 48), stream(96, 144), tiles, lone, dw(1), dw(2), tiles]
    at = lambda i: [(1 << 34) * (5 * i + j + 1) if j != 3 else 0 for j in range(5)]
    fake = FakeList([(k, rec, [a if j != 2 or k.cls != 7 else 0 for j, a in enumerate(at(i))], 0) for i, (k, rec) in enumerate(entries)])
    got = [(l.kernel, l.listed, l.entries, l.tile_m, l.tile_n, l.tile_k) for l in fake.launches()]
    of_lone = api.tt_debug_launch(None, lone[0].cls, lone[0].shape)[0]
    d1, d2 = (api.TT_LISTED_DEPTHWISE, 1, 2, 4, 2, 4), (api.TT_LISTED_DEPTHWISE, 1, 2, 2, 2, 4)
    s = lambda k: (api.TT_LISTED_STREAM, 1, 2, 16, 16, k)
    t = got[6]
    assert t[:3] == (api.TT_LISTED_TILES, 1, 2) and t[3:] != (128, 256, 64)
    assert got == [d1, d2, s(32), s(32), s(96), s(96), t, (api.TT_LISTED_RECORD, 0, 1, of_lone.tile_m, of_lone.tile_n, of_lone.tile_k),
                   d1, d2, t]


@pytest.mark.parametrize("m, n, k, streams", [
    (200704, 24, 32, 1), (50176, 16, 28, 1), (50176, 16, 32, 0), (50176, 20, 40, 0),  # twice the reduction's elements in, one out
    (8192, 96, 16, 1), (8128, 96, 16, 0), (3136, 64, 16, 1), (3136, 64, 20, 0),       # workgroups of 64 rows for half of the CUs
    (50176, 36, 36, 1), (50176, 32, 36, 0), (50176, 64, 36, 0), (50176, 144, 96, 1), (50176, 192, 96, 0), (50176, 144, 100, 0)])
def test_which_contractions_are_streams(m, n, k, streams):
    kernel, rec = wl.Kernel(5, wl.GemmShape(1, m, n, k, 1, wl.F32)), mfma(5, 16, 16, 16, 16, 16, 16, vec=4)
    at = lambda i: [(1 << 34) * (5 * i + j + 1) if j != 3 else 0 for j in range(5)]
    listed = FakeList([(kernel, rec, at(i), 0) for i in range(2)]).launches()
    assert [l.kernel for l in listed] == [api.TT_LISTED_STREAM if streams else api.TT_LISTED_TILES] * 2


# ---- on the GPU -------------------------------------------------------------------------------------------------------
def conv(cls, n, c, h, w, k, f, stride, dtype):
    return wl.Kernel(cls, wl.ConvShape(n, c, h, w, k, f, f, stride, stride, f // 2, f // 2, dtype))


def gemm(cls, m, n, k, dtype, batch=1):
    return wl.Kernel(cls, wl.GemmShape(batch, m, n, k, 1, dtype))


SPLIT = dict(tm=64, tn=64, tk=32, wm=32, wn=32, mf=32, split_k=3, stages=2)
SPLIT_SMALL = dict(tm=16, tn=16, tk=32, wm=16, wn=16, mf=16, split_k=2, stages=2)
LISTS = {
    # ragged in M, N and K, rows that are not whole vectors, residuals, strides, a 5x5, one pixel, every activation
    "bf16": [conv(1, 2, 40, 15, 11, 72, 3, 1, wl.BF16), conv(2, 1, 64, 17, 17, 61, 3, 2, wl.BF16), conv(0, 3, 8, 9, 9, 130, 1, 1, wl.BF16),
             conv(1, 1, 136, 1, 1, 24, 3, 1, wl.BF16), conv(2, 2, 48, 21, 19, 264, 5, 1, wl.BF16), gemm(4, 100, 88, 456, wl.BF16),
             gemm(5, 17, 16, 40, wl.BF16), gemm(6, 130, 261, 328, wl.BF16), gemm(7, 65, 48, 400, wl.BF16, 5), gemm(6, 300, 520, 1032, wl.BF16),
             conv(1, 1, 512, 7, 7, 64, 3, 1, wl.BF16), gemm(4, 40, 40, 2048, wl.BF16)],
    "f32": [conv(1, 2, 36, 15, 11, 72, 3, 1, wl.F32), conv(2, 1, 64, 17, 17, 61, 3, 2, wl.F32), conv(3, 3, 8, 9, 9, 130, 1, 1, wl.F32),
            conv(0, 1, 132, 1, 1, 24, 3, 1, wl.F32), gemm(4, 100, 88, 452, wl.F32), gemm(5, 17, 16, 20, wl.F32), gemm(4, 70, 61, 640, wl.F32),
            conv(1, 1, 512, 7, 7, 64, 3, 1, wl.F32)],
    # large contractions beside small ones
    "bf16_large": [conv(1, 8, 128, 28, 28, 128, 3, 1, wl.BF16)] * 3 + [gemm(6, 1024, 768, 768, wl.BF16)] * 2 +
                  [gemm(4, 520, 3000, 776, wl.BF16), gemm(5, 64, 64, 64, wl.BF16)],
    "f32_large": [conv(2, 2, 64, 28, 28, 128, 3, 1, wl.F32)] * 4 + [gemm(4, 4100, 136, 48, wl.F32), gemm(5, 300, 1032, 96, wl.F32)],
    # the 256 x 256 block kernel, ragged, blocks of 128 rows and columns outside
    "blocks": [gemm(6, 2040, 2040, 1096, wl.BF16)] * 3 + [gemm(5, 1020, 1800, 1096, wl.BF16)] * 2,
    "conv_blocks": [conv(2, 32, 256, 14, 14, 256, 3, 1, wl.BF16)] * 9,
    # depthwise: strides, windows that end outside, one pixel, padding of none and two, channels that are not whole fours
    "depthwise": [wl.Kernel(8, wl.ConvShape(n, c, h, w, c, 3, 3, st, st, pad, pad)) for n, c, h, w, st, pad in
                  ((2, 32, 28, 28, 1, 1), (1, 96, 15, 13, 1, 1), (3, 4, 9, 1, 1, 1), (1, 960, 7, 7, 1, 1), (2, 20, 6, 5, 1, 0), (1, 8, 3, 3, 1, 2),
                   (2, 24, 28, 28, 2, 1), (1, 144, 57, 31, 2, 1), (5, 16, 4, 4, 2, 0), (1, 12, 1, 1, 2, 1), (2, 30, 9, 9, 1, 1), (1, 7, 10, 12, 2, 1))] +
                 [wl.Kernel(8, wl.ConvShape(1, 16, 17, 17, 16, 3, 3, 1, 1, 1, 1))] * 40,
    # streams: every instance's reductions (whole pieces and not), rows and columns that end inside a block, chunks of columns,
    # residuals, every activation; and two entries that are none
    "thin": [gemm(4, 3001, 20, 32, wl.F32), gemm(5, 9001, 96, 16, wl.F32), gemm(4, 130, 20, 20, wl.F32), gemm(4, 17, 16, 16, wl.F32),
             conv(2, 3, 28, 53, 52, 36, 1, 1, wl.F32), conv(3, 2, 24, 65, 64, 44, 1, 1, wl.F32), gemm(5, 3001, 772, 20, wl.F32),
             gemm(5, 40000, 260, 96, wl.F32), conv(2, 2, 36, 65, 64, 44, 1, 1, wl.F32), gemm(4, 8203, 36, 52, wl.F32),
             conv(0, 1, 68, 92, 91, 40, 1, 1, wl.F32), conv(3, 1, 36, 100, 90, 100, 1, 1, wl.F32),
             gemm(4, 1003, 24, 100, wl.F32), gemm(5, 4099, 32, 192, wl.F32)],
    # more entries than a launch takes
    "many": [gemm(5, 20 + 3 * i, 16 + 8 * (i % 5), 40 + 8 * i, wl.BF16) for i in range(43)],
}


def run_list_against_lone_calls(kernels, recs, without_bias=(), oracle_flops=2e8, check=lambda launches: None):
    """Every entry of a list against the same kernel run by itself and, where that is quick, against the oracle."""
    import torch
    import parity as P
    from paper_2201_05587_amd import harness
    inputs = [wl.make_inputs(k, 900 + i) for i, k in enumerate(kernels)]
    dks = [harness.device_kernel(k, 0, inp, max_split=3) for k, inp in zip(kernels, inputs)]
    for i in without_bias:
        tensors = dict(dks[i].tensors)
        del tensors["bias"]
        dks[i] = api.DeviceKernel(kernels[i].cls, kernels[i].shape, tensors, 1, "", dks[i].ws.numel())
    want = []
    for k, dk, r in zip(kernels, dks, recs):
        want.append(P.run_gpu(k, dk, r))
        dk.output().fill_(float("nan"))
        dk.ws.fill_(255)
    listed = api.KernelList(dks, recs)
    launches = listed.launches()
    check(launches)
    listed.run()
    torch.cuda.synchronize()
    for i, (k, dk, w) in enumerate(zip(kernels, dks, want)):
        got = harness.output_in_definition_order(k, dk.output()).float().cpu().numpy()
        P.assert_close(got, w, k.shape.dtype, f"{i} {launches[i].tile_m}x{launches[i].tile_n}")
        if k.flops() < oracle_flops and i not in without_bias:
            P.assert_close(got, P.oracle_output(k, inputs[i]), k.shape.dtype, f"{i} oracle")


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(LISTS))
@pytest.mark.parametrize("split", [False, True])
def test_entries_of_different_shapes_in_shared_launches(name, split):
    kernels = LISTS[name]
    recs = [None] * len(kernels)
    for i, k in enumerate(kernels):
        for fields in (SPLIT, SPLIT_SMALL):
            rec = mfma(k.cls, **fields)
            if split and i % 2 and recs[i] is None and api.tt_schedule_apply(rec, k.cls, k.shape).runnable():
                recs[i] = rec
    if split and name == "depthwise":
        pytest.skip("a depthwise reduction has nine elements: no record splits it")
    assert any(recs) == split

    def check(launches):
        assert len({l.launch for l in launches}) < len(kernels)
        if name.endswith("blocks") and not split:
            assert all(l.tile_m == 256 and l.tile_n == 256 for l in launches)
        if name == "thin" and not split:
            assert [l.kernel for l in launches] == [api.TT_LISTED_STREAM] * 12 + [api.TT_LISTED_TILES] * 2
            assert len({l.launch for l in launches}) == 3
        if name == "depthwise":
            assert [l.listed for l in launches[:12]] == [1] * 10 + [0] * 2 and len({l.launch for l in launches}) == 5

    run_list_against_lone_calls(kernels, recs, without_bias=(0,) if split else (), check=check)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["thin", "depthwise", "f32", "bf16"])
def test_infinities_and_nan_in_shared_launches(name):
    """Elements behind a reduction, outside a window or in another row must not count, whatever they are: the outputs that are
    no numbers are those of the lone calls (an activation takes a NaN to zero there and here), the others are as close."""
    import torch
    import parity as P
    from paper_2201_05587_amd import harness
    kernels = LISTS[name][:12]
    dks = [harness.device_kernel(k, 20 + i, max_split=1) for i, k in enumerate(kernels)]
    for dk in dks:
        x = next(dk.tensors[t] for t in ("x", "a") if t in dk.tensors).view(-1)
        for at, value in ((0, float("inf")), (x.numel() // 3, float("nan")), (x.numel() - 1, float("-inf"))):
            x[at] = value
    want = [P.run_gpu(k, dk) for k, dk in zip(kernels, dks)]
    for dk in dks:
        dk.output().fill_(7.0)
    listed = api.KernelList(dks, [None] * len(dks))
    assert any(l.listed for l in listed.launches())
    listed.run()
    torch.cuda.synchronize()
    special = 0
    for i, (k, dk, w) in enumerate(zip(kernels, dks, want)):
        got = harness.output_in_definition_order(k, dk.output()).float().cpu().numpy()
        for kind in (np.isnan, np.isposinf, np.isneginf):
            np.testing.assert_array_equal(kind(got), kind(w), err_msg=f"{name} {i} {kind.__name__}")
        special += int((~np.isfinite(w)).sum())
        P.assert_close(np.where(np.isfinite(got), got, 0), np.where(np.isfinite(w), w, 0), k.shape.dtype, f"{name} {i}")
    assert special > 0 or name == "depthwise"  # (clamped to six, a NaN to zero)


@pytest.mark.gpu
def test_lists_on_streams_of_their_own_from_threads_of_their_own():
    """Three threads, each with a stream, tensors and workspaces of its own, plan and send their lists at the same time."""
    import threading
    import torch
    import parity as P
    from paper_2201_05587_amd import harness
    names = ("f32", "bf16", "thin")
    dks = [[harness.device_kernel(k, 100 * t + i, max_split=3) for i, k in enumerate(LISTS[n])] for t, n in enumerate(names)]
    recs = [[mfma(k.cls, **SPLIT) if i == 0 and n != "thin" else None for i, k in enumerate(LISTS[n])] for n in names]
    lists = [api.KernelList(d, r) for d, r in zip(dks, recs)]
    want = []
    for l, ds in zip(lists, dks):
        l.run()
        torch.cuda.synchronize()
        want.append([d.output().clone() for d in ds])
    for ds in dks:
        for d in ds:
            d.output().fill_(float("nan"))
    torch.cuda.synchronize()
    failed = []

    def work(l):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                for _ in range(20):
                    l.run()
            stream.synchronize()
        except Exception as e:  # (an assertion in a thread would pass unseen)
            failed.append(e)

    threads = [threading.Thread(target=work, args=(l,)) for l in lists]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
    for n, ds, ws in zip(names, dks, want):
        for i, (d, w) in enumerate(zip(ds, ws)):
            assert torch.equal(d.output(), w), (n, i)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["bf16", "f32", "thin"])
def test_a_list_as_recorded_runs_what_lone_calls_run(name):
    """No two of these entries have one plan, so each has a launch to itself: the same bits."""
    import torch
    import parity as P
    from paper_2201_05587_amd import harness
    kernels = LISTS[name]
    recs = [mfma(k.cls, **SPLIT) if i % 3 == 1 else mfma(k.cls, 16, 16, 16 if k.shape.dtype == wl.F32 else 32, 16, 16, 16, stages=2) if i % 3 == 2 else None
            for i, k in enumerate(kernels)]
    recs = [r if r is None or api.tt_schedule_apply(r, k.cls, k.shape).runnable() else None for k, r in zip(kernels, recs)]
    assert any(recs)
    dks = [harness.device_kernel(k, 60 + i, max_split=3) for i, k in enumerate(kernels)]
    want = [P.run_gpu(k, dk, r) for k, dk, r in zip(kernels, dks, recs)]
    for dk in dks:
        dk.output().fill_(float("nan"))
        dk.ws.fill_(255)
    api.KernelList(dks, recs).run_as_recorded()
    torch.cuda.synchronize()
    for i, (k, dk, w) in enumerate(zip(kernels, dks, want)):
        got = harness.output_in_definition_order(k, dk.output()).float().cpu().numpy()
        np.testing.assert_array_equal(got, w, err_msg=str(i))


def lists_by_tile():
    """The cheapest list of equal entries (ragged in every extent) of a grid of sizes that the rule runs in each of its
    tiles: (data type, convolution?, tile) -> (kernel, count)."""
    best = {}
    for dt in (wl.BF16, wl.F32):
        for is_conv in (True, False):
            for m in (49, 300, 1000, 2000, 6300):
                for n in (24, 136, 264, 520, 1032):
                    for k in (40, 72, 264, 520, 1160):
                        for count in (2, 3, 6):
                            if m * n * k * count > (3e9 if dt == wl.BF16 else 3e8):
                                continue
                            if is_conv:
                                c, hw = max(8, k // 9 // 8 * 8), 7 if m < 300 else 13 if m < 3000 else 29
                                if c * 9 < 0.7 * k:
                                    continue
                                kernel = conv(2, max(1, m // hw // hw), c, hw, hw, n, 3, 1, dt)
                            else:
                                kernel = gemm(5, m + 3, n, k, dt)
                            at = lambda i: [(1 << 34) * (5 * i + j + 1) if j != 3 or is_conv else 0 for j in range(5)]
                            l = FakeList([(kernel, None, at(i), 0) for i in range(count)]).launches()[0]
                            key = (dt, is_conv, l.tile_m, l.tile_n, l.tile_k)
                            if l.listed and (key not in best or best[key][0].flops() * best[key][1] > kernel.flops() * count):
                                best[key] = (kernel, count)
    return best


@pytest.mark.gpu
def test_shared_launches_in_every_tile():
    cases = lists_by_tile()
    assert len(cases) >= 20, sorted(cases)
    for key, (kernel, count) in sorted(cases.items()):
        print(key, kernel.shape, count, flush=True)
        run_list_against_lone_calls([kernel] * count, [None] * count, oracle_flops=1e9,
                                    check=lambda ls: [None for l in ls if (l.tile_m, l.tile_n, l.tile_k) == key[2:]] or 1 / 0)


@pytest.mark.gpu
def test_a_list_replayed_in_a_graph():
    """Shared launches and the second step of split reductions under capture: every replay against the eager pass."""
    import torch
    import parity as P
    from paper_2201_05587_amd import harness
    kernels = LISTS["f32"]
    dks = [harness.device_kernel(k, 70 + i, max_split=3) for i, k in enumerate(kernels)]
    recs = [None] * len(dks)
    recs[0] = mfma(kernels[0].cls, **SPLIT)
    listed = api.KernelList(dks, recs)
    listed.run()
    torch.cuda.synchronize()
    want = [dk.output().cpu().numpy() for dk in dks]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        listed.run()
    for _ in range(3):
        for dk in dks:
            dk.output().fill_(float("nan"))
            dk.ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        for i, (dk, w) in enumerate(zip(dks, want)):
            np.testing.assert_array_equal(dk.output().cpu().numpy(), w, err_msg=str(i))
        listed.run()
        torch.cuda.synchronize()
