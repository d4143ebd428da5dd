"""The unscheduled loop nest: rows shorter than its pieces, reductions that end inside one, every family."""
import pytest

from paper_2201_05587_amd import api
from paper_2201_05587_amd import workloads as wl


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("k", [1, 3, 4, 5, 7, 8, 9, 15, 16, 20, 31])
def test_direct_against_the_oracle(k, dtype):
    import parity as P
    for n in (1, 3, 4, 6, 33):
        for kernel in (wl.Kernel(7, wl.GemmShape(3, 17, n, k, 1, dtype), 1, f"qk_{n}_{k}"), wl.Kernel(7, wl.GemmShape(2, 19, n, k, 0, dtype), 1, f"pv_{n}_{k}"),
                       wl.Kernel(2, wl.ConvShape(2, k, 5, 6, n, 3, 3, 2, 1, 1, 2, dtype), 1, f"conv_{n}_{k}"), wl.Kernel(6, wl.GemmShape(1, 40, n, k, 1, dtype), 1, f"dense_{n}_{k}")):
            direct = api.make_schedule(kernel.cls, api.TT_SK_DIRECT, 1, 1, 1, 1, 1, 0, 1, 0, 1, 1, 1)
            P.check_kernel(kernel, [direct], seed=3 * k + n)


def direct(cls):
    return api.make_schedule(cls, api.TT_SK_DIRECT, 1, 1, 1, 1, 1, 0, 1, 0, 1, 1, 1)


# kernel, entries, outputs of a thread: to either side of the line, of rows shorter than four and of runs shorter than a piece
GRIDS = [(wl.Kernel(7, wl.GemmShape(65, 31, 31, 31, 1, wl.BF16)), 1, 1), (wl.Kernel(7, wl.GemmShape(65, 31, 31, 31, 1, wl.BF16)), 7, 4),
         (wl.Kernel(6, wl.GemmShape(1, 10000, 40, 8, 1, wl.BF16)), 1, 4), (wl.Kernel(6, wl.GemmShape(1, 9999, 40, 8, 1, wl.BF16)), 1, 1),
         (wl.Kernel(6, wl.GemmShape(1, 20000, 37, 7, 1, wl.BF16)), 1, 1), (wl.Kernel(4, wl.GemmShape(1, 20000, 37, 7, 1, wl.F32)), 1, 4),
         (wl.Kernel(7, wl.GemmShape(1, 150000, 3, 40, 1, wl.F32)), 1, 1), (wl.Kernel(7, wl.GemmShape(200, 50, 50, 9, 0, wl.BF16)), 1, 1),
         (wl.Kernel(4, wl.GemmShape(1, 20000, 37, 3, 1, wl.F32)), 1, 1)]


@pytest.mark.parametrize("kernel,count,outputs", GRIDS)
def test_the_grid_of_a_launch(kernel, count, outputs):
    """As launched, which is not the plan's (a workgroup per 256 outputs)."""
    s = kernel.shape
    plan, which = api.tt_debug_launch(direct(kernel.cls), kernel.cls, s, count)
    assert which == api.TT_LAUNCH_RECORD and plan.block == 256
    assert plan.grid == -(-s.batch * s.m * -(-s.n // outputs) // 256)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16])
@pytest.mark.parametrize("k", [8, 9, 20])
def test_four_outputs_a_thread_against_the_oracle(k, dtype):
    import parity as P
    for kernel in (wl.Kernel(7, wl.GemmShape(9, 1200, 39, k, 1, dtype), 1, f"qk_{k}"), wl.Kernel(2, wl.ConvShape(3, k, 45, 46, 66, 3, 3, 1, 1, 1, 1, dtype), 1, f"conv_{k}")):
        assert api.tt_debug_launch(direct(kernel.cls), kernel.cls, kernel.shape)[0].grid < 450  # (400 thousand outputs and more)
        P.check_kernel(kernel, [direct(kernel.cls)], seed=k)
