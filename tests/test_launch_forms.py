"""Which kernels the calls go to, on a runtime that writes it down (tests/recorded.py): the results are the same in every form, so that
no comparison of them tells whether a form was taken."""
import pytest

from recorded import kernels, run

X, Y, NEXT_Y, OUT_X, OUT_Y = (1 << k for k in (43, 44, 45, 46, 47))     # device memory
SAME, BF16, U8 = 0, 1, 2
EXACT, BERNOULLI = 0, 1
UNIFORM, FIFO, RESERVOIR = 0, 1, 2


def forms(calls, selection, classes=300, slots=12, elems=64, storage=SAME, eviction=UNIFORM):
    results = run([["create", classes, slots, elems, storage, selection, eviction, 100], *calls])
    assert all(result == 0 for result, _ in results)
    return [kernels(lines) for _, lines in results[1:]]


# A step of large counts whose labels were announced, and the one they were announced for.
@pytest.mark.parametrize("selection,b,c,r,planned", [
    (EXACT, 4096, 1024, 1024, True), (EXACT, 4096, 1025, 40, False), (EXACT, 4096, 40, 1025, False),
    (BERNOULLI, 1024, 1024, 70, True), (BERNOULLI, 1025, 512, 70, True), (BERNOULLI, 1025, 513, 70, False),
    (BERNOULLI, 4096, 512, 1024, True), (BERNOULLI, 4096, 513, 70, False), (BERNOULLI, 4096, 320, 1, True),
])
def test_announced_steps_of_large_counts(selection, b, c, r, planned):
    calls = [["rb_announce_next", "rb", NEXT_Y], ["rb_update_sample", "rb", X, Y, b, c, r, 1, 0, OUT_X, OUT_Y],
             ["rb_update_sample", "rb", X, NEXT_Y, b, c, r, 1, 1, OUT_X, OUT_Y]]
    _, first, second = forms(calls, selection)
    assert (first == ["rb_big_plan_kernel", "rb_step_big_kernel"] and second == ["rb_step_big_kernel"]) is planned, (first, second)
    if not planned:
        assert first == second == forms([calls[1]], selection)[0]


# Mini-batches of more than 1024 with the Bernoulli selection: not where the plan takes longer than what it saves.
@pytest.mark.parametrize("eviction", [UNIFORM, FIFO, RESERVOIR])
@pytest.mark.parametrize("b,c,r,classes,storage,elems,planned", [
    (2000, 400, 69, 3613, SAME, 64, True), (2000, 400, 69, 3614, SAME, 64, None),          # many classes whose state is kept
    (2000, 300, 69, 4600, U8, 64, True), (2000, 300, 69, 4700, BF16, 64, None),            # ... more with fewer candidates
    (1024, 400, 69, 10240, SAME, 64, True),
    (1171, 36, 12, 7541, BF16, 64, True),                                                  # the other form would be two launches
    (1025, 512, 1, 10240, SAME, 8040, None), (1025, 512, 1, 10240, SAME, 8044, True),      # rows of 6 us
    (2000, 300, 9, 1, SAME, 64, True), (2000, 301, 9, 1, SAME, 64, False),                 # one class of all candidates
    (2000, 301, 1, 1, SAME, 9104, False), (2000, 301, 1, 1, SAME, 9108, True), (2000, 512, 9, 2, BF16, 64, True),
])
def test_announced_steps_of_large_mini_batches_with_coins(b, c, r, classes, storage, elems, planned, eviction):
    _, first, second = forms([["rb_announce_next", "rb", NEXT_Y], ["rb_update_sample", "rb", X, Y, b, c, r, 1, 0, OUT_X, OUT_Y],
                              ["rb_update_sample", "rb", X, NEXT_Y, b, c, r, 1, 1, OUT_X, OUT_Y]], BERNOULLI, classes, 12, elems, storage, eviction)
    assert (second == ["rb_step_big_kernel"]) is (eviction == UNIFORM if planned is None else planned), (first, second)


# Four steps from one call: in one launch (behind the first one's plan), or one by one.
@pytest.mark.parametrize("selection,b,c,together", [(EXACT, 4096, 200, True), (BERNOULLI, 1024, 200, True), (BERNOULLI, 1024, 1024, True),
                                                    (BERNOULLI, 1025, 200, False), (BERNOULLI, 4096, 512, False), (BERNOULLI, 4096, 513, False)])
def test_several_steps_of_large_counts(selection, b, c, together):
    n = 4
    call = ["rb_update_sample_many", "rb", n, [X] * n, [Y + 8 * b * i for i in range(n)], b, c, 70, 1, 0, [OUT_X] * n, [OUT_Y] * n]
    got = forms([call], selection)[0]
    if together:
        assert got[0] == "rb_bigwin_plan_kernel" and set(got[1:]) == {"rb_bigwin_kernel"} and len(got) <= n
    elif c <= 512:
        assert got == ["rb_big_plan_kernel"] + n * ["rb_step_big_kernel"]
    else:
        assert set(got) <= {"rb_step_one_kernel", "rb_update_kernel", "rb_sample_kernel"}


# Where the kernels for many candidates and many representatives begin.
@pytest.mark.parametrize("selection,c", [(EXACT, 64), (EXACT, 65), (EXACT, 192), (EXACT, 193), (EXACT, 4096), (BERNOULLI, 1), (BERNOULLI, 4096)])
def test_updates_of_any_count(selection, c):
    small = selection == EXACT and c <= 64
    assert forms([["rb_update", "rb", X, Y, 4096, c, 1, 0]], selection) == [["rb_update_small_kernel" if small else "rb_update_kernel"]]
