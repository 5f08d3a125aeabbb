"""What a pipeline's calls ask of the two streams, on a runtime that writes it down (tests/recorded.py): orders that results only show
when they go wrong at the right moment."""
import pytest

from recorded import kernels, run

RB_EHIP = -4
BUFFER, TRAIN, OTHER = 100, 200, 300                      # streams
X, Y, OUT_X, OUT_Y = (1 << k for k in (43, 44, 45, 46))    # device memory


def step(at, train, b=64, c=8, r=8):
    return ["rb_pipeline_step", "pipe", X, Y, b, c, r, 1, at, OUT_X, OUT_Y, train]


def step_many(n, at, train, b=64, c=8, r=8):
    return ["rb_pipeline_step_many", "pipe", n, [X] * n, [Y + 8 * b * i for i in range(n)], b, c, r, 1, at, [OUT_X] * n, [OUT_Y] * n, train]


def drain(train):
    return ["rb_pipeline_drain", "pipe", train]


def on_a_pipeline(calls, classes=1000):
    """Results and lines of the calls on a new pipeline of a buffer on stream BUFFER."""
    results = run([["create", classes, 4, 3072, 0, 0, 0, BUFFER], ["rb_pipeline_create"], *calls])
    assert results[0][0] == 0 and results[1][0] == 0
    return results[2:]


def waits_for_the_steps_before(lines, train):
    """Whether, behind these lines in order, stream `train` has waited for an event recorded behind the last launch on BUFFER."""
    behind = {}                                            # event -> launches on BUFFER when it was recorded
    launches = seen = 0
    for line in lines:
        what, *rest = line.split()
        if what == "launch" and rest[1] == str(BUFFER):
            launches += 1
            if len(rest) == 6:
                behind[rest[5]] = launches
        elif what == "record" and rest[1] == str(BUFFER):
            behind[rest[0]] = launches
        elif what == "wait" and rest[0] == str(train):
            seen = max(seen, behind.get(rest[1], 0))
    return launches > 0 and seen == launches


# A call whose training stream is the buffer's own needs no event; whoever has to wait for it from another stream does.
@pytest.mark.parametrize("before", [[], [step(0, TRAIN)], [step_many(4, 0, TRAIN), drain(TRAIN)]], ids=["first", "after-a-step", "after-many"])
@pytest.mark.parametrize("one_stream", [step(4, BUFFER), step_many(4, 4, BUFFER)], ids=["step", "many"])
def test_representatives_collected_on_the_training_stream_are_waited_for_by_another(before, one_stream):
    for then in (drain(TRAIN), step(8, TRAIN), step_many(4, 8, TRAIN)):
        *earlier, (result, last) = on_a_pipeline([*before, one_stream, then, drain(OTHER)])[:-1]
        assert result[0] == 0
        lines = [line for _, some in earlier for line in some]
        # (up to where the call's own steps start)
        first = next((i for i, line in enumerate(last) if line.startswith("launch")), len(last))
        assert waits_for_the_steps_before(lines + last[:first], TRAIN), (lines, last)
    results = on_a_pipeline([*before, one_stream, drain(TRAIN), drain(OTHER)])
    assert waits_for_the_steps_before([line for _, some in results for line in some], OTHER)


def test_a_pipeline_on_one_stream_makes_no_stream_wait():
    for result, lines in on_a_pipeline([step(0, BUFFER), step_many(4, 1, BUFFER), drain(BUFFER)]):
        assert result[0] == 0 and kernels(lines) == [line.split()[1] for line in lines]


def test_the_buffers_next_stream_stands_for_the_one_the_representatives_were_collected_on():
    NEXT = 400                                             # (ordered behind BUFFER by the caller)
    results = on_a_pipeline([step(0, BUFFER), ["rb_set_stream", "rb", NEXT], drain(NEXT), drain(OTHER), step(1, OTHER)])
    assert [lines for _, lines in results[2:4]] == [[], [f"record 2 {NEXT}", f"wait {OTHER} 2"]]
    assert results[4][1][0] == f"wait {OTHER} 2"


CALLS = {
    "update": [["rb_update", "rb", X, Y, 64, 8, 1, 0]],
    "update-general": [["rb_update", "rb", X, Y, 640, 300, 1, 0]],
    "sample": [["rb_sample_augment", "rb", 8, 1, 0, OUT_X, OUT_Y]],
    "sample-general": [["rb_sample_augment", "rb", 80, 1, 0, OUT_X, OUT_Y]],
    "small": [["rb_update_sample", "rb", X, Y, 64, 8, 8, 1, 0, OUT_X, OUT_Y]],
    "one": [["rb_update_sample", "rb", X, Y, 640, 300, 200, 1, 0, OUT_X, OUT_Y]],
    "planned": [["rb_announce_next", "rb", Y], ["rb_update_sample", "rb", X, Y, 64, 8, 8, 1, 0, OUT_X, OUT_Y]],
    "planned-large": [["rb_announce_next", "rb", Y], ["rb_update_sample", "rb", X, Y, 640, 300, 200, 1, 0, OUT_X, OUT_Y]],
    "many": [step_many(4, 0, TRAIN)],
    "many-large": [step_many(4, 0, TRAIN, 640, 300, 200)],
    "bind": [["rb_bind", "rb", 1 << 40, 1 << 41, 1 << 42, BUFFER]],
    "standin": [["rb_standin_compute", BUFFER, X, 4, 1]],
    "copy": [["rb_copy_bytes", BUFFER, X, Y, 4096, 4, 1]],
}


# hipGetLastError tells of any call that has failed on the thread before; what it has to say is neither taken for a launch's nor taken away.
@pytest.mark.parametrize("name", sorted(CALLS))
def test_errors_that_others_have_left_are_left_alone(name):
    *results, pending = on_a_pipeline([["pend", 98], *CALLS[name], ["pending"]])
    last = results[-1][0]
    assert (last[0] if isinstance(last, list) else last) == 0
    assert [r for r in results[1:]] == on_a_pipeline(CALLS[name])
    assert pending[0] == (98 if name != "bind" else 0)     # (rb_bind asks whether memory is the host's, which fails where it is nobody's)


@pytest.mark.parametrize("name", sorted(CALLS))
def test_a_failed_launch_is_reported_once_and_can_be_made_again(name):
    function = "hipExtLaunchKernel" if name.startswith("many") else "hipLaunchKernel"
    *_, (failed, _), pending, _, again = on_a_pipeline([["fail", function, 0], *CALLS[name], ["pending"], ["fail", "", 0], CALLS[name][-1]])
    assert (failed[0] if isinstance(failed, list) else failed) == RB_EHIP and pending[0] == 0
    assert (again[0][0] if isinstance(again[0], list) else again[0]) == 0


# A call that fails on the way may have enqueued a part of its work, and nothing says where that ends: whoever waits next waits for all of it.
@pytest.mark.parametrize("function,after,failing,launched", [
    ("hipEventRecord", 1, step(1, TRAIN), 1),                          # the step is on its way, its event is not
    ("hipEventRecord", 1, step_many(3, 1, TRAIN, 2000, 1100, 40), 3),  # the same for steps that go out one by one
    ("hipLaunchKernel", 1, step(1, TRAIN, 3000, 2, 1500), 1),          # the second of two launches
    ("hipLaunchKernel", 2, step_many(3, 1, TRAIN, 2000, 1100, 40), 2), # the third step of three
    ("hipExtLaunchKernel", 0, step_many(4, 1, TRAIN), 1),              # the last launch of several steps
], ids=["step-event", "many-event", "step-launch", "many-launch", "many-last-launch"])
def test_a_pipeline_call_that_fails_on_the_way_is_waited_for(function, after, failing, launched):
    for before in ([], [step(0, TRAIN)]):
        results = on_a_pipeline([*before, ["fail", function, after], failing, ["fail", "", 0], step(0, TRAIN)], classes=300)
        (result, lines), (again, next_lines) = results[len(before) + 1], results[-1]
        assert result[0] == RB_EHIP and len(kernels(lines)) >= launched, (result, lines)
        assert again[0] == 0
        if before:
            results = on_a_pipeline([*before, ["fail", function, after], failing, ["fail", "", 0], drain(OTHER)], classes=300)
            assert results[-1][0] == [0, 8]                            # the representatives of the last call that succeeded
            assert waits_for_the_steps_before([line for _, some in results for line in some], OTHER), results


# Calls that a stream captures: the buffer's stream joins, no launch carries an event, and the training stream ends up behind all of it.
@pytest.mark.parametrize("call,n", [(step, 1), (step_many, 4)], ids=["step", "many"])
def test_a_captured_pipeline_call_keeps_to_what_a_graph_takes(call, n):
    make = (lambda at: step(at, TRAIN)) if n == 1 else (lambda at: step_many(n, at, TRAIN))
    results = on_a_pipeline([["capture", TRAIN], make(0), make(n), drain(TRAIN), ["end_capture"], make(2 * n)])
    assert [r[0] for r, _ in results[1:4]] == [0, 0, 0] and results[-1][0][0] == 0
    lines = [line for _, some in results[:4] for line in some]
    assert kernels(lines) and all(len(line.split()) == 6 for line in lines if line.startswith("launch"))
    assert lines[:2] == [f"record 1 {TRAIN}", f"wait {BUFFER} 1"] and waits_for_the_steps_before(lines, TRAIN)
    # the second call's steps come behind the wait for the first one's
    second = results[2][1]
    assert second[:3] == [f"wait {TRAIN} 2", f"record 1 {TRAIN}", f"wait {BUFFER} 1"]


# ... and representatives from outside are refused before anything has gone into the graph.
@pytest.mark.parametrize("started", [step(0, TRAIN), step_many(4, 0, TRAIN)], ids=["by-step", "by-many"])
@pytest.mark.parametrize("then", [step(4, TRAIN), step_many(4, 4, TRAIN), drain(TRAIN)], ids=["step", "many", "drain"])
def test_a_capture_takes_no_representatives_from_outside(started, then):
    results = on_a_pipeline([started, ["capture", TRAIN], then, ["pending"], ["end_capture"], then])
    assert results[2][0][0] == RB_EHIP and results[2][1] == [] and results[3][0] == 0
    assert results[-1][0] == [0, 8]
    assert results[-1][1] == on_a_pipeline([started, then])[-1][1]
