"""Arguments of the Python operator calls: what is refused and how, and what stands for a tensor.  Nothing here launches
(the calls that get as far as a plan carry a record of another class)."""
import ctypes

import pytest
import torch

from paper_2201_05587_amd import api
from paper_2201_05587_amd import workloads as wl

CONV = api.to_c_shape(wl.ConvShape(1, 16, 8, 8, 16, 1, 1, 1, 1, 0, 0, wl.F32))
DW = api.to_c_shape(wl.ConvShape(1, 16, 8, 8, 16, 3, 3, 1, 1, 1, 1, wl.F32))
GEMM = api.to_c_shape(wl.GemmShape(1, 16, 16, 16, 1, wl.F32))
OTHER_CLASS = {c: api.make_schedule(wl.CLS_DENSE_ADD if c != wl.CLS_DENSE_ADD else wl.CLS_BATCH_MATMUL)
               for c in (wl.CLS_CONV2D_ADD, wl.CLS_DENSE_ADD, wl.CLS_BATCH_MATMUL, wl.CLS_DWCONV_BIAS_RELU6)}


def tensors(n):
    return [torch.zeros(16 * 16 * 16) for _ in range(n)]


def calls(shape_of=lambda s: s, sched_of=lambda c: OTHER_CLASS[c], first=None, y=True):
    """The four operators on CPU memory, with one argument replaced; `first` stands for x (or a)."""
    x, w, b, out = tensors(4)
    x = first(x) if first else x
    out = out if y else None
    return {
        "conv": lambda: api.tt_conv2d_bias_relu(x, w, b, None, shape_of(CONV), wl.CLS_CONV2D_ADD,
                                                sched_of(wl.CLS_CONV2D_ADD), y=out),
        "dense": lambda: api.tt_dense_bias_relu(x, w, b, shape_of(GEMM), wl.CLS_DENSE_ADD, sched_of(wl.CLS_DENSE_ADD), y=out),
        "matmul": lambda: api.tt_batch_matmul(x, w, shape_of(GEMM), sched_of(wl.CLS_BATCH_MATMUL), c=out),
        "dwconv": lambda: api.tt_dwconv(x, w, b, shape_of(DW), sched_of(wl.CLS_DWCONV_BIAS_RELU6), y=out),
    }


def status(call):
    with pytest.raises(api.TTError) as e:
        call()
    return e.value.status


OPS = ("conv", "dense", "matmul", "dwconv")


@pytest.mark.parametrize("op", OPS)
def test_structures_of_another_type_are_refused(op):
    other = {"conv": GEMM, "dense": CONV, "matmul": CONV, "dwconv": GEMM}[op]
    with pytest.raises(ctypes.ArgumentError):
        calls(shape_of=lambda s: other)[op]()
    with pytest.raises(ctypes.ArgumentError):
        calls(sched_of=lambda c: api.tt_plan())[op]()
    for no_structure in (bytes(200), bytearray(108), {}, 7):
        with pytest.raises(TypeError):
            calls(sched_of=lambda c: no_structure)[op]()


@pytest.mark.parametrize("op", OPS)
def test_structures_of_a_derived_type_are_taken(op):
    class Shape(type(GEMM) if op in ("dense", "matmul") else type(CONV)):
        pass

    class Schedule(api.tt_schedule):
        pass

    def derived(kind, s):
        out = kind()
        ctypes.memmove(ctypes.byref(out), ctypes.byref(s), ctypes.sizeof(s))
        return out

    call = calls(shape_of=lambda s: derived(Shape, s), sched_of=lambda c: derived(Schedule, OTHER_CLASS[c]))[op]
    assert status(call) == api.TT_ERR_CLASS_MISMATCH


@pytest.mark.parametrize("op", OPS)
def test_missing_tensors(op):
    assert status(calls(first=lambda x: None)[op]) == api.TT_ERR_BAD_ARG
    with pytest.raises(AttributeError):  # nothing says what the output should be
        calls(first=lambda x: None, y=False)[op]()


class Memory:
    """Device memory of a caller's own: all a call asks of an argument is where it lies."""

    def __init__(self, t, shift=0):
        self.t, self.shift = t, shift
        self.dtype, self.device = t.dtype, t.device

    def data_ptr(self):
        return self.t.data_ptr() + self.shift


@pytest.mark.parametrize("op", OPS)
def test_whatever_has_a_data_ptr_is_taken(op):
    for y in (True, False):
        assert status(calls(first=Memory, y=y)[op]) == api.TT_ERR_CLASS_MISMATCH
        assert status(calls(first=lambda t: Memory(t, 4), y=y)[op]) == api.TT_ERR_BAD_ARG  # not 16-byte aligned
    with pytest.raises(AttributeError):
        calls(first=lambda t: [1.0, 2.0])[op]()
