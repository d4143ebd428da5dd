"""Depthwise launches in windows: every window and channel count of a thread, at maps that the windows do not divide."""
import numpy as np
import pytest

from paper_2201_05587_amd import api, harness
from paper_2201_05587_amd import workloads as wl


def kernel(n, c, h, w, stride, pad=1):
    return wl.Kernel(wl.CLS_DWCONV_BIAS_RELU6, wl.ConvShape(n, c, h, w, c, 3, 3, stride, stride, pad, pad, wl.F32), 1, f"dw_{n}_{c}_{h}x{w}_s{stride}_p{pad}")


# (n, c, h, w, stride, pad), the window it runs in and the channels of a thread: maps of one output to more than a workgroup's,
# pieces to either side of every line of the rule, padding wider than the window
CASES = [((1, 1, 8, 8, 1, 1), (1, 1, 1)), ((3, 5, 7, 9, 1, 1), (1, 1, 1)), ((2, 6, 8, 5, 2, 1), (1, 1, 2)), ((1, 64, 3, 3, 1, 0), (1, 1, 4)),
         ((1, 4, 5, 6, 1, 4), (1, 1, 4)), ((1, 1, 256, 256, 1, 1), (1, 1, 1)), ((1, 1, 256, 257, 1, 1), (1, 2, 1)), ((1, 2, 511, 515, 2, 1), (1, 2, 2)),
         ((3, 44, 89, 91, 1, 1), (1, 2, 4)), ((1, 3, 131, 1001, 1, 0), (1, 2, 1)), ((1, 1, 512, 769, 1, 1), (2, 2, 1)), ((2, 2, 901, 907, 2, 1), (2, 2, 2)),
         ((5, 28, 107, 113, 1, 1), (2, 2, 4)), ((1, 4, 1499, 1601, 2, 0), (2, 2, 4)), ((1, 3, 1399, 1249, 1, 1), (2, 2, 1)),
         ((1, 3, 1401, 1251, 1, 1), (4, 2, 1)), ((2, 2, 2293, 2299, 1, 1), (4, 2, 2)), ((1, 4, 2291, 2303, 1, 2), (4, 2, 4))]
RECORDS = [(8, 8, 4, 2, 2, 1), (2, 8, 16, 1, 4, 4), (7, 8, 8, 7, 1, 2)]  # tile_m, tile_n, tile_k, wave_m, wave_n, vec


def base(k, stages=1):
    """The default record, which names outputs one by one, in `stages`."""
    r = api.tt_schedule_default(k.cls, k.shape)
    assert r.sketch == api.TT_SK_DWCONV
    r.stages = stages
    return r


@pytest.mark.parametrize("case,window", CASES)
def test_the_rule_of_windows(case, window):
    k = kernel(*case)
    plan, which = api.tt_debug_launch(None, k.cls, k.shape)
    assert which == api.TT_LAUNCH_RECORD and (plan.wave_m, plan.wave_n, plan.eff_vec_a) == window
    threads = k.shape.n * k.shape.c // window[2] * -(-k.shape.ho // window[0]) * -(-k.shape.wo // window[1])
    assert plan.block == 256 and plan.grid * 256 >= threads and plan.grid % 8 == 0
    assert api.launched_name(None, k.cls, k.shape) == f"tt::dwconv3x3_window_kernel<{case[4]}, {window[2]}, {window[0]}, {window[1]}>"
    # an LDS patch is the record's
    assert api.launched_name(base(k, 2), k.cls, k.shape).startswith("tt::dwconv3x3_kernel")


@pytest.mark.gpu
@pytest.mark.parametrize("case,window", CASES)
def test_windows_against_the_oracle(case, window):
    """As the default and under records of other tiles (the same launch); nothing is written behind the output."""
    import torch

    from parity import assert_close, oracle_output
    k = kernel(*case)
    inp = wl.make_inputs(k, 11)
    ref = oracle_output(k, inp)
    dk = harness.device_kernel(k, 11, inp)
    out = dk.output()
    room = torch.empty(out.numel() + 64, device="cuda")
    dk.desc.bufs[3] = room.data_ptr()
    recs = [api.make_schedule(k.cls, api.TT_SK_DWCONV, tm, tn, tk, wm, wn, 0, 1, 0, v, 1, 1) for tm, tn, tk, wm, wn, v in RECORDS]
    recs = [r for r in recs if api.tt_schedule_apply(r, k.cls, k.shape).runnable()]
    for rec in [None] + recs[:1 if out.numel() > 1 << 20 else None]:
        room.fill_(-77.0)
        assert dk.run(rec) == api.TT_OK
        torch.cuda.synchronize()
        got = harness.output_in_definition_order(k, room[:out.numel()].view(out.shape)).cpu().numpy()
        assert_close(got, ref, wl.F32, f"{k.name} {rec}")
        assert bool((room[out.numel():] == -77.0).all())


@pytest.mark.gpu
@pytest.mark.parametrize("case", [(2, 12, 9, 11, 1), (2, 7, 9, 11, 2), (3, 32, 60, 61, 1)])
def test_entries_of_one_plan(case):
    """Up to eight entries of a list under its records go out as rows of one launch."""
    import torch
    k = kernel(*case)
    dks = [harness.device_kernel(k, 20 + i) for i in range(11)]
    api.KernelList(dks, [None] * len(dks)).run_as_recorded()
    torch.cuda.synchronize()
    together = [dk.output().clone() for dk in dks]
    for dk, got in zip(dks, together):
        dk.output().fill_(float("nan"))
        assert dk.run(None) == api.TT_OK
        torch.cuda.synchronize()
        assert torch.equal(dk.output(), got)
    assert not torch.equal(together[0], together[1])


REFUSED, VALID = (16, 7, 64, 1, 7, 4), (8, 8, 16, 1, 2, 4)  # (the first names 1024 threads of seven outputs)


@pytest.mark.gpu
def test_a_search_counts_no_refused_record():
    """Records that the operator refuses share no time with those that run in the same windows."""
    k = kernel(4, 256, 56, 56, 1)
    pool = [api.make_schedule(k.cls, api.TT_SK_DWCONV, tm, tn, tk, wm, wn, 0, 1, 0, v, 1, 1) for tm, tn, tk, wm, wn, v in (REFUSED, VALID)]
    dk = harness.device_kernel(k, 3)
    assert dk.run(pool[0]) == api.TT_ERR_UNSUPPORTED and dk.run(pool[1]) == api.TT_OK
    opts = api.tt_sweep_opts(warmup=1, samples=3, min_sample_us=20, max_launches=4, allow_slower_than_default=1)
    rows, us, _, _ = api.tt_transfer_sweep([dk], pool, opts)
    assert us[0][0] == -1 and us[0][1] > 0
    assert (rows[0]["chosen"], rows[0]["n_valid"], rows[0]["n_invalid"]) == (1, 1, 1)
