"""What the compiler has made of the kernels: properties of the built device code that their timing rests on and that no result
shows.  Reads the library that was built here."""
import os
import re
import shutil
import subprocess

import pytest

import paper_2406_03285_amd as rb

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
SAME, BF16, U8 = rb.RB_STORE_SAME, rb.RB_STORE_BF16, rb.RB_STORE_U8


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """(kernel, template arguments) -> its instructions in the order they stand in memory."""
    where = tmp_path_factory.mktemp("code")
    lib = shutil.copy(rb.LIB_PATH, where / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, cwd=where, stdout=subprocess.DEVNULL)
    device, = [f for f in os.listdir(where) if f.endswith("gfx950")]
    text = subprocess.Popen([OBJDUMP, "-d", "--mcpu=gfx950", "--no-show-raw-insn", device], cwd=where, stdout=subprocess.PIPE, text=True)
    found, at = {}, None
    for line in text.stdout:
        if line[0] == "\t":
            if at is not None:
                at.append(line.split("//")[0].strip())
        elif line.endswith(">:\n"):
            m = re.search(r"\d(rb_[a-z_]+_kernel)I((?:L[bi]\d+E)+)E", line)
            at = found.setdefault((m[1], tuple(int(v) for v in re.findall(r"L[bi](\d+)E", m[2]))), []) if m else None
    assert text.wait() == 0 and found
    return found


def vmcnt(instruction):
    return instruction.startswith("s_waitcnt") and "vmcnt" in instruction


def most_together(instructions, load):
    """Most loads of one kind behind each other without a wait for any of them."""
    most = run = 0
    for i in instructions:
        if vmcnt(i):
            run = 0
        elif i.startswith(load):
            run += 1
            most = max(most, run)
    return most


@pytest.mark.parametrize("kernel", ["rb_step_big_kernel", "rb_step_planned_kernel", "rb_window_kernel"])
def test_vectors_that_are_converted_at_the_load_are_requested_together(kernels, kernel):
    """A lane of a tile of U vectors kept as bfloat16 (8 bits) has 2 U (4 U) binary32 vectors in flight."""
    seen = 0
    for (name, args), code in kernels.items():
        if name == kernel and args[2] != SAME:
            unroll, storage = args[0], args[2]
            seen += 1
            assert most_together(code, "buffer_load_dwordx4") >= (4 if storage == U8 else 2) * unroll, (name, args)
    assert seen >= 4


def test_sampling_draws_are_made_while_the_counts_travel(kernels):
    """rb_sample_small_kernel: the ten rounds of the draw (two multiplications each; the scalar part of the first rounds is shared)
    stand before the scan of the counts; behind it only the reduction to the range and addresses are left."""
    seen = 0
    for (name, args), code in kernels.items():
        if name == "rb_sample_small_kernel":
            seen += 1
            scan = next(i for i, c in enumerate(code) if "row_shr:1 " in c)
            wide = [i for i, c in enumerate(code) if re.match(r"v_mad_u64_u32|v_mul_(hi|lo)_u32", c)]
            assert sum(i < scan for i in wide) >= 14, (name, args)
    assert seen >= 10


def test_candidates_of_converted_rows_are_placed_while_their_row_travels(kernels):
    """rb_update_small_kernel: the class's count comes from LDS by an LDS access (a flat one waits for every load in flight)."""
    seen = 0
    for (name, args), code in kernels.items():
        if name == "rb_update_small_kernel" and args[2] != SAME:
            seen += 1
            assert not any(c.startswith("flat_load") for c in code), (name, args)
    assert seen >= 12
