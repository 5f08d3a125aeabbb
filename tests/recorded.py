"""Runs calls of the library on a HIP runtime that only writes down what it is asked for (tests/hip_recorder): which kernels go to
which stream, what is recorded and waited for, and what a failing runtime call leaves behind.  No GPU, nothing is computed.

`run(calls)` carries them out in a process of its own, in which the recorder stands in front of the real runtime, and returns
[(result, lines)] of them.  A call is a list: the function's name and its arguments ("rb", "pipe": the handles made last; a list: an
array of device pointers), or one of

    ["create", classes, slots, elems, storage, selection, eviction, stream]   makes and binds a buffer
    ["fail", hip_function, after]      its calls fail, after so many that succeed; "" ends that
    ["pend", error], ["pending"]       a call of somebody else's has failed before; the error that hipGetLastError would tell of
    ["capture", stream], ["end_capture"]
"""
import ctypes as C
import json
import os
import re
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = os.path.join(ROOT, "tests", "hip_recorder", "hip_recorder.c")
LIB = os.environ.get("RB_LIBRARY") or os.path.join(ROOT, "paper_2406_03285_amd", "librb.so")


def run(calls):
    with tempfile.TemporaryDirectory() as where:
        recorder = os.path.join(where, "librecorder.so")
        subprocess.run(["gcc", "-std=c11", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", SOURCE, "-o", recorder], check=True)
        out = subprocess.run([sys.executable, os.path.abspath(__file__), recorder], input=json.dumps(calls), capture_output=True, text=True)
    assert out.returncode == 0, (out.returncode, out.stderr)
    return [(result, lines) for result, lines in json.loads(out.stdout)]


def kernels(lines):
    """Names of the kernels among the lines."""
    return [line.split()[1] for line in lines if line.startswith("launch")]


def _child(recorder, calls):
    R = C.CDLL(recorder, mode=C.RTLD_GLOBAL)             # before the library, and so before the runtime it is linked to
    R.recorder_lines.restype = C.c_char_p
    L = C.CDLL(LIB)
    u64 = C.c_uint64
    handles = {"rb": 0, "pipe": 0}

    def call(name, *args):
        kept = []
        for a in args:
            if isinstance(a, str):
                kept.append(u64(handles[a]))
            elif isinstance(a, list):
                kept.append((u64 * len(a))(*a))
            else:
                kept.append(u64(a or 0))
        return getattr(L, name)(*kept)

    results = []
    for name, *args in calls:
        R.recorder_clear()
        if name == "fail":
            R.recorder_fail(args[0].encode(), args[1])
            result = 0
        elif name == "pend":
            R.recorder_pend(args[0])
            result = 0
        elif name == "pending":
            result = R.recorder_pending()
        elif name == "capture":
            R.recorder_capture(u64(args[0]))
            result = 0
        elif name == "end_capture":
            R.recorder_end_capture()
            result = 0
        elif name == "create":
            classes, slots, elems, storage, selection, eviction, stream = args
            h, shape = C.c_void_p(), (C.c_int64 * 1)(elems)
            result = L.rb_create(C.byref(h), C.c_int64(classes), C.c_int64(slots), shape, 1, 0)
            handles["rb"] = h.value
            result = result or call("rb_set_storage", "rb", storage) or call("rb_set_policy", "rb", selection, eviction)
            result = result or call("rb_bind", "rb", 1 << 40, 1 << 41, 1 << 42, stream)
        elif name == "rb_pipeline_create":
            h = C.c_void_p()
            result = L.rb_pipeline_create(C.byref(h), C.c_void_p(handles["rb"]))
            handles["pipe"] = h.value
        elif name in ("rb_pipeline_step", "rb_pipeline_step_many", "rb_pipeline_drain", "rb_query_steps_per_launch", "rb_query_launches"):
            number = C.c_int64(-1)
            result = [call(name, *args, C.addressof(number)), number.value]
        else:
            result = call(name, *args)
        lines = [re.sub(r"launch \S*\d(rb_[a-z_]+_kernel)\S*", r"launch \1", line) for line in R.recorder_lines().decode().splitlines()]
        results.append((result, lines))
    return results


if __name__ == "__main__":
    print(json.dumps(_child(sys.argv[1], json.load(sys.stdin))))
