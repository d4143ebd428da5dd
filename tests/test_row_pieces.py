"""Epilogues of outputs whose rows are no whole 16-byte vectors: every remainder of a row, in every kernel that writes a tile."""
import numpy as np
import pytest

from paper_2201_05587_amd import api, harness
from paper_2201_05587_amd import workloads as wl

GUARD = 64  # elements behind the output


def record(cls, dtype, stages, tm, tn, wm, wn, mfma=16, split_k=1):
    bf16 = dtype == wl.BF16
    return api.make_schedule(cls, api.TT_SK_MFMA, tm, tn, 64 if bf16 else 32, wm, wn, mfma, split_k, 1, 8 if bf16 else 4, 8, stages)


# register pipeline and ring, waves of two and of four bands, blocks of 32, two splits, one tile (which a reduction of 640
# sends out in groups)
RECORDS = [(2, 64, 64, 32, 32, 16, 1), (3, 64, 64, 32, 32, 16, 1), (3, 64, 64, 32, 32, 32, 1), (3, 32, 32, 16, 16, 16, 2), (3, 128, 64, 32, 32, 16, 1)]


def kernels(dtype, n, k):
    yield wl.Kernel(wl.CLS_BATCH_MATMUL, wl.GemmShape(2, 129, n, k, 1, dtype), 1, f"qk_{n}_{k}")
    yield wl.Kernel(wl.CLS_DENSE_BIAS_GELU if dtype == wl.BF16 else wl.CLS_DENSE_BIAS_RELU, wl.GemmShape(1, 130, n, k, 1, dtype), 1, f"dense_{n}_{k}")
    yield wl.Kernel(wl.CLS_CONV2D_BIAS_ADD_RELU, wl.ConvShape(1, k, 11, 13, n, 1, 1, 1, 1, 0, 0, dtype), 1, f"res_{n}_{k}")
    yield wl.Kernel(wl.CLS_CONV2D_BIAS_RELU6, wl.ConvShape(1, 16, 9, 15, n, 3, 3, 1, 1, 1, 1, dtype), 1, f"conv_{n}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 9, 31, 33, 62, 63, 65, 66, 67, 100, 131])
def test_every_remainder_of_a_row(n, dtype):
    """Against the oracle; nothing is written behind the output."""
    import torch

    from parity import assert_close, oracle_output
    ran = 0
    for k in (128, 640):
        for kernel in kernels(dtype, n, k):
            inp = wl.make_inputs(kernel, 7)
            ref = oracle_output(kernel, inp)
            dk = harness.device_kernel(kernel, 7, inp)
            size = dk.output().numel()
            room = torch.empty(size + GUARD, dtype=dk.output().dtype, device="cuda")
            where = [i for i in range(5) if dk.desc.bufs[i] == dk.output().data_ptr()]
            assert len(where) == 1
            dk.desc.bufs[where[0]] = room.data_ptr()
            for stages, tm, tn, wm, wn, mfma, split in RECORDS:
                rec = record(kernel.cls, dtype, stages, tm, tn, wm, wn, mfma, split)
                if not api.tt_schedule_apply(rec, kernel.cls, kernel.shape).runnable():
                    continue  # (a tile wider than the row)
                room.fill_(-77.0)
                rc = dk.run(rec)
                torch.cuda.synchronize()
                assert rc == api.TT_OK, (api.status_name(rc), kernel.name, rec)
                out = room[:size].view(dk.output().shape)
                assert_close(harness.output_in_definition_order(kernel, out).float().cpu().numpy(), ref, dtype, f"{kernel.name} {rec}")
                assert bool((room[size:] == -77.0).all()), (kernel.name, rec)
                ran += 1
            room.fill_(-77.0)
            rc = dk.run(None)
            torch.cuda.synchronize()
            assert rc == api.TT_OK
            assert_close(harness.output_in_definition_order(kernel, room[:size].view(dk.output().shape)).float().cpu().numpy(), ref, dtype, kernel.name)
            assert bool((room[size:] == -77.0).all()), kernel.name
    assert ran or n < 32
