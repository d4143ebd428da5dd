"""What operator calls launch, without a GPU: launches([(cls, shape, record or None), ...]) makes the calls in one process of
their own, in order, on top of launch_recorder.cpp, and returns (status, launches) of each."""
import ctypes
import dataclasses
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))


def launches(calls):
    with tempfile.TemporaryDirectory() as tmp:
        lib = os.path.join(tmp, "recorder.so")
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-o", lib, os.path.join(HERE, "launch_recorder.cpp")])
        asked = [(cls, dataclasses.asdict(shape), None if rec is None else rec.knobs()) for cls, shape, rec in calls]
        out = subprocess.run([sys.executable, os.path.abspath(__file__), lib], input=json.dumps(asked), capture_output=True, text=True,
                             cwd=os.path.dirname(HERE), timeout=300)
    assert out.returncode == 0, out.stderr
    return json.loads(out.stdout.splitlines()[-1])


def main():
    recorder = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # ahead of the runtime that the library brings
    recorder.recorded_name.restype = ctypes.c_char_p
    sys.path.insert(0, os.path.dirname(HERE))
    from paper_2201_05587_amd import api
    from paper_2201_05587_amd import workloads as wl
    answers = []
    for cls, shape, knobs in json.load(sys.stdin):
        recorder.forget()
        k = wl.Kernel(cls, (wl.ConvShape if "stride_h" in shape else wl.GemmShape)(**shape))
        s, rec = api.to_c_shape(k.shape), None if knobs is None else api.make_schedule(**knobs)
        r, p = rec and ctypes.byref(rec), 4096  # (no launch reads it)
        if cls == wl.CLS_DWCONV_BIAS_RELU6:
            rc = api.lib.tt_dwconv(p, p, p, p, ctypes.byref(s), r, None)
        elif k.is_conv():
            rc = api.lib.tt_conv2d_bias_relu(p, p, p, p if cls == wl.CLS_CONV2D_BIAS_ADD_RELU else None, p, ctypes.byref(s), cls, r, p, 1 << 40, None)
        elif cls == wl.CLS_BATCH_MATMUL:
            rc = api.lib.tt_batch_matmul(p, p, p, ctypes.byref(s), r, p, 1 << 40, None)
        else:
            rc = api.lib.tt_dense_bias_relu(p, p, p, p, ctypes.byref(s), cls, r, p, 1 << 40, None)
        made = []
        for i in range(recorder.recorded()):
            n = (ctypes.c_uint * 5)()
            recorder.recorded_shape(i, n)
            made.append(dict(name=recorder.recorded_name(i).decode(), grid=n[0], entries=n[1], block=n[2], lds=n[3], enabled=n[4]))
        answers.append((rc, made))
    print(json.dumps(answers))


if __name__ == "__main__":
    main()
