"""CPU-side checks of the C-ABI library: it loads, exports every function the
header declares, and rejects bad arguments on the host before any device work."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "rb.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(rb_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_function():
    import paper_2406_03285_amd as rb
    names = _declared()
    assert len(names) >= 10 and set(names) == set(rb.EXPORTS)
    lib = C.CDLL(rb.LIB_PATH)
    for name in names:
        assert getattr(lib, name) is not None


def test_binding_has_the_same_names():
    import paper_2406_03285_amd as rb
    for name in _declared():
        assert callable(getattr(rb, name))


@pytest.mark.parametrize("layout", ["hp", "hiiipp", "hppiiii", "hppiiiiipp"])
def test_native_marshalling_passes_what_ctypes_passes(layout):
    """Integers of any size, None, tensors, bools, floats, numpy numbers, keywords, wrong counts and types."""
    import numpy as np
    import torch
    from paper_2406_03285_amd import binding
    ctype = {"h": C.c_void_p, "p": C.c_void_p, "i": C.c_int64}
    seen = []
    entry = C.CFUNCTYPE(C.c_int, *[C.c_uint64] * len(layout))(lambda *a: seen.append(a) or len(a) - 5)
    through_ctypes = C.cast(entry, C.CFUNCTYPE(C.c_int, *[ctype[k] for k in layout]))
    names = [f"a{i}" for i in range(len(layout))]

    def general(*args, **kw):
        args = args + tuple(kw[n] for n in names[len(args):])
        return through_ctypes(*[binding._ptr(v) if k == "p" else int(v) if k == "i" else v for v, k in zip(args, layout, strict=True)])

    native = binding.Call(C.cast(entry, C.c_void_p).value, layout, general)
    t = torch.zeros(4)
    usual = {"h": 2 ** 47 + 8, "p": 2 ** 46 + 16, "i": 5}
    odd = {"h": [None, 0, 7, C.c_void_p(9), 3.5], "p": [None, 0, t, True, 3.5, object()],
           "i": [0, -1, 2 ** 63, 2 ** 64 - 1, 2 ** 64 + 3, -2 ** 70, True, 2.75, np.int64(-4), np.float32(2.0), torch.tensor(6), "8", None, []]}
    cases = [(tuple(usual[k] for k in layout), {})]
    for i, k in enumerate(layout):
        cases += [(tuple(v if j == i else usual[q] for j, q in enumerate(layout)), {}) for v in odd[k]]
    cases += [(cases[0][0][:-1], {}), (cases[0][0] + (1,), {}), (cases[0][0][:1], dict(zip(names[1:], cases[0][0][1:])))]
    for args, kw in cases:
        got = []
        for f in (native, general):
            seen.clear()
            try:
                got.append((f(*args, **kw), list(seen)))
            except Exception as e:      # noqa: BLE001  (the same refusal from both)
                got.append((type(e), list(seen)))
        assert got[0] == got[1], (args, kw)
    assert native.__wrapped__ is general and native.__name__ == "general"


@pytest.mark.parametrize("name", ["rb_announce_next_many", "rb_update_sample_many", "rb_pipeline_step_many", "rb_pipeline_drain"])
def test_native_marshalling_of_many_steps_passes_what_ctypes_passes(name, monkeypatch):
    """Lists and tuples of addresses and tensors of the right and of other lengths, pointer arrays, None, what is neither, streams."""
    import inspect
    import torch
    from paper_2406_03285_amd import binding
    native = getattr(binding, name)
    general = native.__wrapped__
    params = list(inspect.signature(general).parameters)
    kinds = ["v" if q in ("batch_x", "batch_y", "out_x", "out_y", "next_x", "next_y", "next_batch_y") else "s" if q == "train_stream" else
             "h" if q in ("rb", "p") else "i" for q in params]
    rows = name.startswith("rb_pipeline")
    seen = []

    def entry(*a):
        n = a[1] if "v" in kinds else 0
        seen.append([[(C.c_uint64 * n).from_address(v)[:n] if v else None] if k == "v" else v for v, k in zip(a, kinds)])
        if rows:
            C.c_int64.from_address(a[len(kinds)]).value = -3
        return 7

    function = C.CFUNCTYPE(C.c_int, *[C.c_uint64] * (len(kinds) + rows))(entry)
    ctype = {"h": C.c_void_p, "v": C.POINTER(C.c_void_p), "i": C.c_int64, "s": C.c_void_p}
    through_ctypes = C.cast(function, C.CFUNCTYPE(C.c_int, *[ctype[k] for k in kinds], *[C.POINTER(C.c_int64)] * rows))

    class Library:
        pass

    setattr(Library, name, staticmethod(through_ctypes))
    monkeypatch.setattr(binding, "_L", Library)
    there = binding.Call(C.cast(function, C.c_void_p).value, "".join(kinds), general, rows)

    class Stream:
        def __init__(self, v):
            self.cuda_stream = v

    t = torch.zeros(4)
    usual = {"h": 2 ** 47 + 8, "i": 3, "v": [2 ** 46 + 16, t, 0], "s": 2 ** 45}
    odd = {"h": [None, 0, 3.5], "i": [-1, 2 ** 64 + 3, True, 2.75, None], "s": [None, 0, -1, Stream(0), Stream(2 ** 44), Stream(True), 2.5],
           "v": [None, (1, 2, t), [1, None, True], [2 ** 64 + 5, -1, 1], [1, 2, 3.5], [1, 2, object()], binding.pointer_array([4, 5, t]), 5, "abc",
                 range(3), [1, 2, 3, 4]]}
    cases = [(tuple(usual[k] for k in kinds), {})]
    for i, k in enumerate(kinds):
        if k == "i" and params[i] == "n":
            continue                                    # (as many as there are items)
        cases += [(tuple(v if j == i else usual[q] for j, q in enumerate(kinds)), {}) for v in odd[k]]
    if "v" in kinds:
        for n in (0, 1, 64, 65):
            cases.append((tuple([8 * i for i in range(n)] if k == "v" else n if q == "n" else usual[k] for q, k in zip(params, kinds)), {}))
    cases += [(cases[0][0][:-1], {}), (cases[0][0] + (1,), {}), (cases[0][0][:1], dict(zip(params[1:], cases[0][0][1:])))]
    for args, kw in cases:
        got = []
        for f in (there, general):
            seen.clear()
            try:
                got.append((f(*args, **kw), list(seen)))
            except Exception as e:      # noqa: BLE001  (the same refusal from both)
                got.append((type(e), list(seen)))
        assert got[0] == got[1], (args, kw)
    assert native.__name__ == name


@pytest.mark.parametrize("name", ["rb_update", "rb_sample_augment", "rb_update_sample", "rb_announce_next", "rb_bind"])
def test_calls_are_copied_pickled_referenced_and_bound_like_functions(name):
    import copy
    import inspect
    import pickle
    import weakref
    import paper_2406_03285_amd as rb
    f = getattr(rb, name)
    for protocol in range(pickle.HIGHEST_PROTOCOL + 1):
        assert pickle.loads(pickle.dumps(f, protocol)) is f
    assert copy.copy(f) is f and copy.deepcopy([f]) == [f]
    assert weakref.ref(f)() is f
    f.note = [name]
    try:
        assert f.note == [name] and f.__dict__["note"] == [name] and vars(f)["note"] == [name]
    finally:
        del f.note
    assert not hasattr(f, "note")
    assert f.__name__ == name and f.__module__ == "paper_2406_03285_amd.binding" and f.__doc__ is None
    assert f.__get__(None, object) is f and next(iter(inspect.signature(f).parameters)) == "rb"

    class Handle(int):          # a handle that carries its calls as methods
        call = f

    missing = [0] * (len(inspect.signature(f).parameters) - 1)
    assert Handle(0).call(*missing) == f(0, *missing) == rb.RB_EINVAL


@pytest.mark.parametrize("error", [KeyboardInterrupt, MemoryError, AttributeError, TypeError, RuntimeError])
def test_what_data_ptr_raises_ends_the_call(error):
    """... as it does in the Python function: once asked, nothing called, the very exception handed on."""
    import paper_2406_03285_amd as rb
    asked = []

    class Sample:
        def data_ptr(self):
            asked.append(error("first" if not asked else "again"))
            if len(asked) > 1:
                return 16
            raise asked[0]

    for f in (rb.rb_announce_next, rb.rb_announce_next.__wrapped__):
        asked.clear()
        with pytest.raises(error) as caught:
            f(0, Sample())
        assert len(asked) == 1 and caught.value is asked[0]


def test_a_call_object_without_a_function_raises():
    import subprocess
    import sys
    code = """
from paper_2406_03285_amd._calls import Call
c = Call.__new__(Call)
def refuses(error, f):
    try:
        f()
    except error:
        return
    raise SystemExit(f"{error} expected")
refuses(AttributeError, lambda: c.__wrapped__)
refuses(AttributeError, lambda: c.__name__)
refuses(AttributeError, lambda: c.__reduce__())
refuses(TypeError, lambda: c(1, 2))
refuses(ValueError, lambda: c.__init__(0, "hp", len))
refuses(TypeError, lambda: c(1, 2))
assert c.__doc__ is None
"""
    done = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert done.returncode == 0, (done.returncode, done.stderr[-500:])


def test_without_the_native_marshalling_the_calls_go_through_ctypes():
    """Where Python's headers are missing the extension cannot be built: the package works all the same."""
    import subprocess
    import sys
    code = """
import sys
sys.modules["paper_2406_03285_amd._calls"] = None       # an import of it raises ModuleNotFoundError
import types
import paper_2406_03285_amd as rb
for name in ("rb_update", "rb_sample_augment", "rb_update_sample", "rb_announce_next"):
    assert isinstance(getattr(rb, name), types.FunctionType), name
assert rb.rb_update(None, None, None, 1, 1, 0, 0) == rb.RB_EINVAL
"""
    done = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert done.returncode == 0, (done.returncode, done.stderr[-500:])


def test_the_native_marshalling_is_built_here_and_for_this_interpreter():
    import sysconfig
    from paper_2406_03285_amd import _calls, build
    assert _calls.__file__ == build.CALLS and build.CALLS.endswith(sysconfig.get_config_var("EXT_SUFFIX"))


def test_create_validation_and_sizes():
    import paper_2406_03285_amd as rb
    rc, h = rb.rb_create(1000, 130, (3, 224, 224), rb.RB_F32)
    assert rc == rb.RB_OK and h
    rc, xb, yb, wb = rb.rb_query_sizes(h)
    assert rc == rb.RB_OK and xb == 1000 * 130 * 602112 and yb == 1000 * 130 * 8 and wb % 256 == 0 and wb < (4 << 20)
    # hot calls before rb_bind
    assert rb.rb_update(h, 256, 256, 4, 2, 0, 0) == rb.RB_ESTATE
    assert rb.rb_sample_augment(h, 2, 0, 0, 256, 256) == rb.RB_ESTATE
    # argument errors are reported before the state error
    assert rb.rb_update(h, None, 256, 4, 2, 0, 0) == rb.RB_EINVAL
    assert rb.rb_update(h, 256, 256, 0, 0, 0, 0) == rb.RB_EINVAL            # b < 1
    assert rb.rb_update(h, 256, 256, 4, 5, 0, 0) == rb.RB_EINVAL            # c > b
    assert rb.rb_update(h, 256, 256, 4, -1, 0, 0) == rb.RB_EINVAL
    assert rb.rb_update(h, 256, 256, rb.RB_MAX_BATCH + 1, 1, 0, 0) == rb.RB_EINVAL
    assert rb.rb_update(h, 264, 256, 4, 2, 0, 0) == rb.RB_EINVAL            # batch_x not 16-byte aligned
    assert rb.rb_sample_augment(h, -1, 0, 0, 256, 256) == rb.RB_EINVAL
    assert rb.rb_sample_augment(h, rb.RB_MAX_BATCH + 1, 0, 0, 256, 256) == rb.RB_EINVAL
    assert rb.rb_sample_augment(h, 2, 0, 0, None, 256) == rb.RB_EINVAL
    assert rb.rb_bind(h, None, 256, 256) == rb.RB_EINVAL
    assert rb.rb_bind(h, 256, 256, 128) == rb.RB_EINVAL                     # workspace not 256-byte aligned
    assert rb.rb_set_option(h, rb.RB_OPT_UNROLL, 3) == rb.RB_EINVAL
    assert rb.rb_set_option(h, rb.RB_OPT_UNROLL, 4) == rb.RB_OK
    assert rb.rb_set_option(h, 99, 0) == rb.RB_EINVAL
    assert rb.rb_destroy(h) == rb.RB_OK


@pytest.mark.parametrize("args", [
    (0, 10, (4,), 0), (10, 0, (4,), 0), (10, 10, (), 0), (10, 10, (3,), 0),      # 12-byte row
    (10, 10, (4,), 7), (10, 10, (4, 0), 0), ((1 << 20) + 1, 1, (4,), 0), (1 << 20, 1 << 12, (4,), 0),
    (10, 10, (4,), 1),                                                            # bf16: 8-byte row
])
def test_create_rejects(args):
    import paper_2406_03285_amd as rb
    rc, h = rb.rb_create(*args)
    assert rc == rb.RB_EINVAL and not h


def test_strerror():
    import paper_2406_03285_amd as rb
    assert rb.rb_strerror(0) == "ok"
    assert len({rb.rb_strerror(s) for s in (0, -1, -2, -3, -4, -99)}) == 6


def test_variant_setters_validate_on_the_host():
    import paper_2406_03285_amd as rb
    rc, h = rb.rb_create(4, 2, (8,), rb.RB_F32)
    assert rc == rb.RB_OK
    assert rb.rb_set_policy(h, 2, 0) == rb.RB_EINVAL and rb.rb_set_policy(h, 0, 3) == rb.RB_EINVAL
    assert rb.rb_set_policy(h, rb.RB_SELECT_BERNOULLI, rb.RB_EVICT_RESERVOIR) == rb.RB_OK
    assert rb.rb_set_policy(None, 0, 0) == rb.RB_EINVAL
    assert rb.rb_set_storage(h, 2) == rb.RB_EINVAL and rb.rb_set_storage(None, 0) == rb.RB_EINVAL
    assert rb.rb_query_sizes(h)[1] == 4 * 2 * 32
    assert rb.rb_set_storage(h, rb.RB_STORE_BF16) == rb.RB_OK
    assert rb.rb_query_sizes(h)[1] == 4 * 2 * 16                     # stored rows are half the sample
    assert rb.rb_set_storage(h, rb.RB_STORE_SAME) == rb.RB_OK
    assert rb.rb_query_sizes(h)[1] == 4 * 2 * 32
    rb.rb_destroy(h)
    rc, h = rb.rb_create(4, 2, (8,), rb.RB_BF16)
    assert rb.rb_set_storage(h, rb.RB_STORE_BF16) == rb.RB_EINVAL    # only binary32 samples can be narrowed
    rb.rb_destroy(h)
    rc, h = rb.rb_create(4, 2, (4,), rb.RB_F32)
    assert rb.rb_set_storage(h, rb.RB_STORE_BF16) == rb.RB_EINVAL    # a stored row would be 8 bytes
    rb.rb_destroy(h)
    # the pipeline and the multi-step call reject what the host can see
    assert rb.rb_pipeline_create(None)[0] == rb.RB_EINVAL
    assert rb.rb_pipeline_step(None, 256, 256, 4, 2, 2, 0, 0, 256, 256)[0] == rb.RB_EINVAL
    assert rb.rb_pipeline_drain(None)[0] == rb.RB_EINVAL
    assert rb.rb_pipeline_destroy(None) == rb.RB_EINVAL
    assert rb.rb_update_sample_many(None, 1, [256], [256], 4, 2, 2, 0, 0, [256], [256]) == rb.RB_EINVAL
    # announcements: only host-visible checks, nothing is dereferenced
    rc, h = rb.rb_create(4, 2, (8,), rb.RB_F32)
    assert rb.rb_announce_next(None, 256) == rb.RB_EINVAL and rb.rb_announce_next(h, 4) == rb.RB_EINVAL
    assert rb.rb_announce_next(h, 256) == rb.RB_OK and rb.rb_announce_next(h, None) == rb.RB_OK
    assert rb.rb_announce_next_many(None, 1, [256]) == rb.RB_EINVAL
    assert rb.rb_announce_next_many(h, -1, [256]) == rb.RB_EINVAL
    assert rb.rb_announce_next_many(h, 2, [256, 4]) == rb.RB_EINVAL          # misaligned
    assert rb.rb_announce_next_many(h, 2, [256, 0]) == rb.RB_EINVAL          # null
    assert rb.rb_announce_next_many(h, 1, None) == rb.RB_EINVAL
    assert rb.rb_announce_next_many(h, 12, [256 * (i + 1) for i in range(12)]) == rb.RB_OK
    assert rb.rb_announce_next_many(h, 0, None) == rb.RB_OK
    # steps per launch of the multi-step call: host arithmetic only
    assert rb.rb_query_steps_per_launch(None, 8, 2, 2)[0] == rb.RB_EINVAL
    assert rb.rb_query_steps_per_launch(h, 0, 0, 0)[0] == rb.RB_EINVAL and rb.rb_query_steps_per_launch(h, 8, 9, 2)[0] == rb.RB_EINVAL
    # (32-byte samples: rows move sooner than one workgroup plans a step, so the form with two planners per step is chosen)
    assert rb.rb_query_steps_per_launch(h, 64, 8, 8) == (rb.RB_OK, 16) and rb.rb_query_steps_per_launch(h, 512, 64, 64) == (rb.RB_OK, 16)
    assert rb.rb_set_option(h, rb.RB_OPT_PLANNERS, 3) == rb.RB_EINVAL and rb.rb_set_option(h, rb.RB_OPT_PLANNERS, -1) == rb.RB_EINVAL
    assert rb.rb_set_option(h, rb.RB_OPT_PLANNERS, 2) == rb.RB_OK and rb.rb_query_steps_per_launch(h, 64, 8, 8) == (rb.RB_OK, 16)
    assert rb.rb_set_option(h, rb.RB_OPT_PLANNERS, 1) == rb.RB_OK                 # one planner workgroup per launch:
    assert rb.rb_query_steps_per_launch(h, 64, 8, 8) == (rb.RB_OK, 32)            # few rows per step: the most
    assert rb.rb_query_steps_per_launch(h, 512, 64, 64) == (rb.RB_OK, 10)         # 1280 table entries / 128 rows per step
    assert rb.rb_query_steps_per_launch(h, 512, 40, 24) == (rb.RB_OK, 16)         # 640 planner slots / max(c, r)
    assert rb.rb_query_steps_per_launch(h, 512, 65, 8) == (rb.RB_OK, 16)          # beyond the small form: the large-count form's 16
    assert rb.rb_query_steps_per_launch(h, 4096, 8, 8) == (rb.RB_OK, 16)
    assert rb.rb_query_steps_per_launch(h, 4096, 1025, 8) == (rb.RB_OK, 1)        # not eligible for either
    assert rb.rb_query_steps_per_launch(h, 64, 0, 8) == (rb.RB_OK, 1)
    assert rb.rb_set_option(h, rb.RB_OPT_WINDOW, 5) == rb.RB_OK and rb.rb_query_steps_per_launch(h, 64, 8, 8) == (rb.RB_OK, 5)
    assert rb.rb_set_option(h, rb.RB_OPT_WINDOW, 33) == rb.RB_EINVAL
    assert rb.rb_set_policy(h, rb.RB_SELECT_EXACT, rb.RB_EVICT_FIFO) == rb.RB_OK and rb.rb_query_steps_per_launch(h, 64, 8, 8) == (rb.RB_OK, 5)
    assert rb.rb_set_policy(h, rb.RB_SELECT_BERNOULLI, rb.RB_EVICT_FIFO) == rb.RB_OK and rb.rb_query_steps_per_launch(h, 64, 8, 8) == (rb.RB_OK, 5)   # the large-count form takes it
    assert rb.rb_query_steps_per_launch(h, 1025, 8, 8) == (rb.RB_OK, 1)         # ... for mini-batches of at most 1024
    assert rb.rb_query_steps_per_launch(h, 1025, 400, 25) == (rb.RB_OK, 1) and rb.rb_query_steps_per_launch(h, 1024, 400, 25) == (rb.RB_OK, 5)
    rb.rb_destroy(h)
    # the library's choice between the two forms follows the time a step's rows take to move
    rc, h = rb.rb_create(10, 4, (3, 224, 224), rb.RB_F32)
    assert rb.rb_query_steps_per_launch(h, 64, 8, 8) == (rb.RB_OK, 32)            # 16 rows of 602 KB: one planner workgroup keeps up
    assert rb.rb_query_steps_per_launch(h, 64, 4, 4) == (rb.RB_OK, 16)            # 8 rows: it would not
    assert rb.rb_set_option(h, rb.RB_OPT_PLANNERS, 2) == rb.RB_OK and rb.rb_query_steps_per_launch(h, 64, 8, 8) == (rb.RB_OK, 16)
    assert rb.rb_set_option(h, rb.RB_OPT_PLANNERS, 1) == rb.RB_OK and rb.rb_query_steps_per_launch(h, 64, 4, 4) == (rb.RB_OK, 32)
    rb.rb_destroy(h)


def test_launches_of_a_step_validate_on_the_host():
    import paper_2406_03285_amd as rb
    rc, h = rb.rb_create(100, 20, (3072,), rb.RB_F32)
    assert rb.rb_query_launches(None, 8, 2, 2)[0] == rb.RB_EINVAL
    assert rb.rb_query_launches(h, 0, 0, 0)[0] == rb.RB_EINVAL and rb.rb_query_launches(h, 8, 9, 2)[0] == rb.RB_EINVAL
    assert rb.rb_query_launches(h, 8, 2, rb.RB_MAX_BATCH + 1)[0] == rb.RB_EINVAL
    assert rb.rb_query_launches(h, 128, 16, 16) == (rb.RB_OK, 1) and rb.rb_query_launches(h, 256, 100, 90) == (rb.RB_OK, 1)
    assert rb.rb_query_launches(h, 128, 0, 16) == (rb.RB_OK, 1) and rb.rb_query_launches(h, 128, 0, 0) == (rb.RB_OK, 0)
    assert rb.rb_set_option(h, rb.RB_OPT_FUSE, 0) == rb.RB_OK
    assert rb.rb_query_launches(h, 128, 16, 16) == (rb.RB_OK, 2) and rb.rb_query_launches(h, 256, 100, 90) == (rb.RB_OK, 2)
    rb.rb_destroy(h)


# The single launch for any counts adds a step's candidates to the fill counts in 32 bits: a class may hold up to
# slots_per_class samples, and a step offers it up to RB_MAX_BATCH more.
@pytest.mark.parametrize("storage,elems", [(0, 4), (1, 8), (2, 16)], ids=["same", "bf16", "u8"])
@pytest.mark.parametrize("selection", [0, 1])
@pytest.mark.parametrize("eviction", [0, 1, 2])
def test_single_launch_leaves_room_for_a_step_above_the_slots(storage, elems, selection, eviction):
    import paper_2406_03285_amd as rb
    most = 2**31 - 1 - rb.RB_MAX_BATCH
    for classes, slots, launches in ((1, most, 1), (1, most + 1, 2), (1, 2**31 - 1, 2), (2, 2**30 - 1, 1)):
        rc, h = rb.rb_create(classes, slots, (elems,), rb.RB_F32)
        assert rc == rb.RB_OK and rb.rb_set_storage(h, storage) == rb.RB_OK
        assert rb.rb_set_policy(h, selection, eviction) == rb.RB_OK
        for b, c, r in ((4096, 64, 4096), (100, 64, 65), (1, 1, 65)):
            assert rb.rb_query_launches(h, b, c, r) == (rb.RB_OK, launches), (classes, slots, b, c, r)
        rb.rb_destroy(h)


# Few classes: beyond so many candidates of each class per step, what a representative's search among them costs exceeds a launch.
@pytest.mark.parametrize("eviction,classes,most", [(0, 1, 448), (0, 2, 896), (0, 9, 4032), (0, 10, 4096),
                                                   (1, 1, 64), (1, 4, 256), (1, 10, 1120), (1, 20, 3840), (1, 21, 4096),
                                                   (2, 1, 64), (2, 4, 256), (2, 10, 1120), (2, 20, 3840), (2, 21, 4096)])
@pytest.mark.parametrize("selection", [0, 1])
def test_single_launch_with_few_classes(eviction, classes, most, selection):
    import paper_2406_03285_amd as rb
    rc, h = rb.rb_create(classes, 200, (256,), rb.RB_F32)
    assert rb.rb_set_policy(h, selection, eviction) == rb.RB_OK
    for c in (most - 1, most, most + 1, 4096):
        if c <= 4096:
            assert rb.rb_query_launches(h, 4096, c, 100) == (rb.RB_OK, 1 if c <= most else 2), c
    rb.rb_destroy(h)


# Many classes: the single launch reads all fill counts in many workgroups.  Shapes next to the crossing that was measured, on
# both sides of it (what lies far from it on either side is in the same list).
@pytest.mark.parametrize("storage,selection,classes,c,r,launches", [
    (0, 0, 2000, 5, 5, 1), (0, 0, 4000, 5, 5, 1), (0, 0, 5076, 17, 7, 2), (0, 0, 6000, 5, 5, 2), (0, 0, 6000, 30, 30, 1), (0, 0, 8000, 30, 30, 2),
    (0, 0, 6000, 109, 29, 1), (0, 0, 7832, 109, 29, 2), (0, 0, 8000, 200, 200, 1), (0, 0, 10000, 200, 200, 2), (0, 0, 10240, 400, 400, 1),
    (0, 1, 6000, 5, 5, 1), (0, 1, 8000, 5, 5, 2), (0, 1, 8000, 109, 29, 1), (0, 1, 10000, 109, 29, 2), (0, 1, 10240, 200, 200, 1),
    (1, 0, 2000, 5, 5, 1), (1, 0, 6000, 5, 5, 2), (1, 0, 8000, 30, 30, 2), (1, 0, 8000, 200, 200, 1), (1, 0, 10240, 400, 400, 1),
    (1, 1, 6000, 5, 5, 1), (1, 1, 10000, 109, 29, 2),
    (2, 0, 2000, 5, 5, 1), (2, 0, 6000, 5, 5, 2), (2, 0, 6000, 30, 30, 2), (2, 0, 6000, 200, 200, 2), (2, 0, 8000, 400, 400, 2),
    (2, 0, 4000, 200, 200, 1), (2, 0, 4000, 400, 400, 1), (2, 0, 9700, 1000, 1000, 1),
    (2, 1, 8000, 5, 5, 2), (2, 1, 6000, 30, 30, 1), (2, 1, 10000, 30, 30, 2), (2, 1, 10240, 400, 400, 1),
    (0, 0, 10241, 1000, 1000, 2), (0, 1, 10241, 1000, 1000, 2),
])
def test_single_launch_with_many_classes(storage, selection, classes, c, r, launches):
    import paper_2406_03285_amd as rb
    rc, h = rb.rb_create(classes, 10, (784,), rb.RB_F32)
    assert rb.rb_set_storage(h, storage) == rb.RB_OK and rb.rb_set_policy(h, selection, 0) == rb.RB_OK
    assert rb.rb_query_launches(h, 4096, c, r) == (rb.RB_OK, launches)
    rb.rb_destroy(h)


# Rows that take too long to move for a launch of one workgroup per compute unit; two launches of the small-count kernels move
# long rows better than those of the general kernels.
@pytest.mark.parametrize("storage,selection,c,r,elems,launches", [
    (0, 0, 56, 21, 48000, 1), (0, 0, 30, 30, 92768, 2), (0, 0, 64, 64, 48000, 2), (0, 0, 60, 10, 92768, 2), (0, 0, 21, 56, 92768, 2),
    (0, 0, 70, 60, 48000, 1), (0, 0, 100, 90, 48000, 1), (0, 0, 120, 100, 48000, 2), (0, 1, 30, 30, 92768, 1), (0, 1, 64, 64, 48000, 1),
    (1, 0, 30, 30, 48000, 1), (1, 0, 64, 64, 48000, 2), (1, 1, 3, 40, 92768, 2), (1, 1, 40, 3, 92768, 1), (1, 0, 10, 60, 48000, 1), (2, 0, 60, 10, 20000, 1), (2, 0, 64, 64, 48000, 2),
])
def test_single_launch_with_long_rows(storage, selection, c, r, elems, launches):
    import paper_2406_03285_amd as rb
    rc, h = rb.rb_create(1378, 4, (elems,), rb.RB_F32)
    assert rb.rb_set_storage(h, storage) == rb.RB_OK and rb.rb_set_policy(h, selection, 0) == rb.RB_OK
    assert rb.rb_query_launches(h, 400, c, r) == (rb.RB_OK, launches)
    rb.rb_destroy(h)


# ... and either side of where the time the rows take, or the representatives' rows, ends it: few or many candidates, either selection.
@pytest.mark.parametrize("storage,selection,c,r,us,launches", [
    (0, 0, 128, 66, 13.9, 1), (0, 0, 128, 66, 14.1, 2), (0, 0, 129, 66, 44.5, 2), (0, 0, 129, 10, 44.5, 1), (0, 0, 129, 10, 45.5, 2),
    (0, 0, 300, 200, 34.0, 1), (0, 0, 300, 200, 36.0, 2), (0, 0, 1025, 1024, 35.5, 1), (0, 0, 1025, 1024, 36.5, 2),
    (0, 0, 1025, 1025, 13.9, 1), (0, 0, 1025, 1025, 14.1, 2), (0, 1, 10, 119, 19.0, 1), (0, 1, 10, 119, 20.0, 2), (0, 1, 119, 10, 44.5, 1),
    (0, 1, 119, 10, 45.5, 2), (0, 1, 64, 64, 13.9, 1), (0, 1, 64, 64, 14.1, 2),
    (1, 0, 65, 195, 7.9, 1), (1, 0, 65, 195, 8.1, 2), (1, 0, 195, 65, 19.8, 1), (1, 0, 195, 65, 20.2, 2), (1, 0, 1025, 1024, 23.5, 1), (1, 0, 1025, 1024, 24.5, 2),
    (1, 1, 32, 97, 10.5, 1), (1, 1, 32, 97, 10.8, 2), (1, 1, 4, 124, 3.35, 1), (1, 1, 4, 124, 3.5, 2),
    (2, 0, 195, 65, 3.9, 1), (2, 0, 195, 65, 4.1, 2), (2, 0, 50, 200, 3.7, 1), (2, 0, 50, 200, 3.8, 2), (2, 0, 1025, 1024, 15.8, 1), (2, 0, 1025, 1024, 16.2, 2),
    (2, 1, 100, 50, 5.4, 1), (2, 1, 100, 50, 5.6, 2), (2, 1, 64, 64, 1.9, 1), (2, 1, 64, 64, 2.1, 2),
])
def test_single_launch_ends_with_the_time_the_rows_take(storage, selection, c, r, us, launches):
    import paper_2406_03285_amd as rb
    elems = int(us * 5.5e6 / (c + r) / (8, 6, 5)[storage]) // 16 * 16
    rc, h = rb.rb_create(1378, 4, (elems,), rb.RB_F32)
    assert rb.rb_set_storage(h, storage) == rb.RB_OK and rb.rb_set_policy(h, selection, 0) == rb.RB_OK
    assert rb.rb_query_launches(h, 2000, c, r) == (rb.RB_OK, launches)
    rb.rb_destroy(h)


# ... converted rows beyond the nearer lines: as many slots as candidates and 32 classes at least.
@pytest.mark.parametrize("storage,elems", [(1, 32000), (2, 13000)])
@pytest.mark.parametrize("classes,slots,launches", [(32, 7, 1), (31, 7, 2), (32, 6, 2), (39, 5, 1), (194, 1, 2), (195, 1, 1)])
def test_single_launch_of_converted_rows_needs_slots(storage, elems, classes, slots, launches):
    import paper_2406_03285_amd as rb
    rc, h = rb.rb_create(classes, slots, (elems // 16 * 16,), rb.RB_F32)
    assert rb.rb_set_storage(h, storage) == rb.RB_OK
    assert rb.rb_query_launches(h, 400, 195, 65) == (rb.RB_OK, launches)
    rb.rb_destroy(h)


def test_single_launch_with_more_representatives_than_slots():
    import paper_2406_03285_amd as rb
    for selection in (0, 1):
        rc, h = rb.rb_create(9, 40, (32,), rb.RB_F32)
        assert rb.rb_set_policy(h, selection, 0) == rb.RB_OK
        for r, launches in ((65, 1), (360, 1), (361, 2), (4096, 2)):
            assert rb.rb_query_launches(h, 100, 9, r) == (rb.RB_OK, launches)
        rb.rb_destroy(h)
    rc, h = rb.rb_create(2, 3, (32,), rb.RB_F32)
    assert rb.rb_query_launches(h, 100, 9, 64) == (rb.RB_OK, 1)             # small counts: one launch in any case
    rb.rb_destroy(h)
