"""The kernels switch the fp32 rounding mode in inline assembly (quot8_truncated, lean_T in mxq_device.hpp).  The
target wants two wait states between two writes of one hardware register, and the compiler, which inserts them between
its own, does not look into inline assembly: the listing of the kernels is checked instead."""
import os
import re
import subprocess

from paper_2605_08565_amd import build

OPEN, CLOSE = "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 3", "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 0"


def writes(listing):
    """(kernel, instruction, wait states before it inside its basic block, instructions since the last write) of every
    write of a hardware register.  An instruction is one wait state, s_nop n is n + 1."""
    kernel, waits, between = None, 0, []
    for line in listing.splitlines():
        text = line.split(";")[0].strip()
        label = re.fullmatch(r"([\w$.]+):", text)
        if label:
            kernel, waits = (label.group(1), 0) if not label.group(1).startswith(".") else (kernel, 0)
            between.append("label")
        elif text and not text.startswith("."):
            op = text.split()[0]
            if op.startswith("s_setreg"):
                yield kernel, " ".join(text.split()), waits, between
                waits, between = 0, []
                continue
            between.append(op)
            waits = 0 if op.startswith(("s_cbranch", "s_branch", "s_setpc", "s_swappc")) else \
                waits + (int(text.split()[1], 0) + 1 if op == "s_nop" else 1)


def test_reader_of_listings():
    text = "k:\n\ts_nop 1\n\ts_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 3\n\tv_mul_f32 v0, v1, v2 ; x\n.LBB0_1:\n\ts_waitcnt 0\n" \
           "\ts_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 0\n"
    assert [(w[0], w[2]) for w in writes(text)] == [("k", 2), ("k", 1)]


def test_writes_of_the_mode_register_are_apart(tmp_path):
    """Counted inside the basic block of the later write, so whatever path leads there; and between the write that opens
    a section and the one that closes it there is nothing but its products."""
    out = str(tmp_path / "stream.s")
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "stream_kernels.hip"), "-o", out],
                   check=True, capture_output=True)
    n, want = 0, OPEN
    for kernel, text, waits, between in writes(open(out).read()):
        assert text == want, (kernel, text)
        assert waits >= 2, (kernel, text, waits)
        if want == CLOSE:
            assert set(between) == {"v_mul_f32_e32"} or set(between) == {"v_mul_f32"}, (kernel, between)
        n, want = n + 1, CLOSE if want == OPEN else OPEN
    assert n > 200 and want == OPEN


def test_only_the_streaming_kernels_write_it():
    users = [f for f in sorted(os.listdir(build.CSRC)) if "s_setreg" in open(os.path.join(build.CSRC, f)).read()]
    assert users == ["mxq_device.hpp"]
    for f in build.SOURCES:
        text = open(os.path.join(build.CSRC, f)).read()
        assert f == "stream_kernels.hip" or not re.search(r"quot8_truncated|lean_T\(", text), f
