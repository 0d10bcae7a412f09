"""What the pruned scale search rests on, checked on the CPU.

A scale S with 3.5 S >= amax never has a lower block SSE than S / 2 where S / 2 is a scale code too
(from code 16 on, and for the even codes below), so the search stops there.  Checked against the
oracle's SSE of every code, in its pinned fp32 arithmetic, together with the set of codes the search
visits: the lowest code of minimal SSE must always be among them.  And the element quotient the search
forms from the hardware reciprocal."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

from paper_2605_08565_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = shutil.which("amdclang++") or "/opt/rocm/llvm/bin/clang++"


def blocks(kind, b, n, rng):
    if kind == "student":
        return (rng.standard_t(4, size=(n, b)) * 0.02).astype(np.float32)
    if kind == "tiny":                                     # scales in the sub-normal codes
        return (rng.standard_normal((n, b)) * 2.0 ** rng.integers(-18, -4, (n, 1))).astype(np.float32)
    # abs-max and elements on grid points and ties of some scale
    s = (1 + rng.integers(0, 8, (n, 1)) / 8.0) * 2.0 ** rng.integers(-10, 4, (n, 1))
    v = rng.integers(0, 15, (n, b)) * 0.25 * s
    v[:, 0] = rng.choice([3.5, 4.0, 5.0, 6.0], n) * s[:, 0]
    return v.astype(np.float32)


@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("b", [2, 4, 16])
@pytest.mark.parametrize("kind", ["student", "tiny", "grid"])
def test_half_scale_dominates_and_walk_finds_the_winner(oracle, fmt, b, kind):
    rng = np.random.default_rng(17 * fmt + b + len(kind))
    top = oracle.scale_max_code(fmt)
    scale = np.array([oracle.scale_decode(fmt, c) for c in range(top + 1)])
    for v in blocks(kind, b, 40, rng):
        sse = np.array([oracle.block_sse(v, fmt, c)[1] for c in range(top + 1)], np.float32)
        amax = float(np.abs(v).max())
        codes = np.arange(1, top + 1)
        has_half = (codes >= 16) | (codes % 2 == 0)
        half = np.where(codes >= 16, codes - 8, codes // 2)
        dominated = has_half & (3.5 * scale[codes] >= amax)
        assert (scale[half[has_half]] * 2 == scale[codes[has_half]]).all()
        assert (sse[half[dominated]] <= sse[codes[dominated]]).all()

        start = max(int(oracle.quantize(v.reshape(1, b), b, fmt, 0)[1][0, 0]), 1)
        best = sse[start]
        seen = {start}
        for c in codes[start:]:                            # upwards: what is not dominated, up to 4 amax
            if not dominated[c - 1] and (c < 16 or 3.5 * scale[c] < amax) and scale[c - 1] < 4 * amax:
                seen.add(int(c))
                best = min(best, sse[c])
        for c in range(start - 1, 0, -1):                  # downwards until the clipping bound exceeds the best
            over = np.float32(amax) - np.float32(6.0) * np.float32(scale[c])
            if over > 0 and np.float32(over * over) > best:
                break
            seen.add(c)
            best = min(best, sse[c])
        assert 1 + int(np.argmin(sse[1:])) in seen, (kind, b, fmt)


@pytest.mark.parametrize("off", [-2, -1, 0, 1, 2])
def test_one_product_gives_the_sse_of_8_bit_inputs(off):
    """bf16 elements without a per-tensor scale: rounding v * r, r within two ulps of 1 / S, leaves the
    residual of the exact quotient, for every significand of v and S (sub-normal codes included)."""
    grid = np.array([0, .5, 1, 1.5, 2, 3, 4, 6])
    mids = (grid[1:] + grid[:-1]) / 2
    v = (np.arange(128, 256)[:, None] * 2.0 ** np.arange(-14, 0)).ravel()
    for s in [1, 3, 5, 7, *range(8, 16)]:
        S = s / 8.0
        r = np.float32(1 / S)
        r = (r.view(np.uint32) + np.uint32(off & 0xFFFFFFFF)).view(np.float32)
        y = (v.astype(np.float32) * r).astype(np.float64)
        for k in (1.0, -1.0):                              # an exact tie may fall either way
            near = np.searchsorted(mids, y + k * 2.0 ** -40, side="left")
            exact = np.min(np.abs(v[:, None] - grid * S), axis=1)
            assert (np.abs(v - grid[near] * S) == exact).all(), (s, off)


def test_quotient_from_hardware_reciprocal(tmp_path):
    if "fma" not in open("/proc/cpuinfo").read():
        pytest.skip("host CPU has no FMA instruction")
    exe = str(tmp_path / "reciprocal_check")
    subprocess.run([CLANG, "-O2", "-std=c++17", "-ffp-contract=off", "-mfma", "-Wall", "-Werror",
                    os.path.join(HERE, "host", "reciprocal_check.cpp"), "-o", exe, "-lm"], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(res.stdout)
    assert res.returncode == 0 and "bad=0" in res.stdout


def test_walk_over_single_blocks_with_the_kernels_rules(tmp_path):
    """The kernel's order of steps over the scalar rules it includes (mxq_arith.hpp): same winner and same
    SSE bits as all codes tried, and never many candidates -- also for blocks beyond the format, which
    the clipping bound of one element alone would send through every code (126 and 254), and for NaN and
    infinity.  The longest way down before a floor is looked for is 16 steps; with the start and the floor
    itself that is 18 candidates; ordinary blocks end well before (15 on these inputs)."""
    if "fma" not in open("/proc/cpuinfo").read():
        pytest.skip("host CPU has no FMA instruction")
    exe = str(tmp_path / "search_walk_check")
    subprocess.run([CLANG, "-O2", "-std=c++17", "-ffp-contract=off", "-mfma", "-Wall", "-Werror",
                    os.path.join(HERE, "host", "search_walk_check.cpp"), "-o", exe, "-lm"], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(res.stdout)
    rows = [dict(t.split("=") for t in l.split()[1:]) for l in res.stdout.splitlines() if "cases=" in l]
    assert res.returncode == 0 and len(rows) == 16
    for r in rows:
        assert int(r["cases"]) > 100 and int(r["bad"]) == 0 and int(r["most"]) <= 18, r


def test_window_over_single_blocks_with_the_kernels_rules(tmp_path):
    """Of the same blocks, those that the window takes: it tries eight codes, one above, the 15 of the 16 steps down that
    are not among the eight, and the floor, 25 at most, where it goes on down behind the window (33 to 35 if it walked from
    its start again).  And the scales under which the kernel takes squares for exact are above 1/512 of the abs-max, as
    exact squares need."""
    if "fma" not in open("/proc/cpuinfo").read():
        pytest.skip("host CPU has no FMA instruction")
    exe = str(tmp_path / "search_walk_check")
    subprocess.run([CLANG, "-O2", "-std=c++17", "-ffp-contract=off", "-mfma", "-Wall", "-Werror",
                    os.path.join(HERE, "host", "search_walk_check.cpp"), "-o", exe, "-lm"], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(res.stdout)
    rows = [dict(t.split("=") for t in l.split()[1:]) for l in res.stdout.splitlines() if "cases=" in l]
    assert res.returncode == 0 and len(rows) == 16
    for r in rows:
        assert int(r["bad"]) == 0 and int(r["most_on"]) <= 25 and float(r["far"]) < 512.0, r
    assert sum(int(r["on"]) for r in rows) > 40 and sum(int(r["window"]) for r in rows) > 20000


def test_search_rules_are_defined_once():
    """In the header that the host check compiles, not a second time in a kernel file."""
    csrc = os.path.join(os.path.dirname(HERE), "paper_2605_08565_amd", "csrc")
    names = ("walk_scale_bias(uint32_t", "walk_halved(uint32_t", "walk_last_odd(float", "saturation_loss(float", "walk_patience(int", "make_recip_from(float")
    for f in os.listdir(csrc):
        text = open(os.path.join(csrc, f)).read()
        assert all((n in text) == (f == "mxq_arith.hpp") for n in names), f


def test_window_rules_are_defined_once():
    csrc = os.path.join(os.path.dirname(HERE), "paper_2605_08565_amd", "csrc")
    for f in os.listdir(csrc):
        text = open(os.path.join(csrc, f)).read()
        assert all((n in text) == (f == "mxq_arith.hpp") for n in ("window_first(uint32_t start, uint32_t", "window_steps(int")), f


def test_pruned_search_kernels_leave_room_for_wavefronts(tmp_path):
    """The search waits for its own instructions' results, so it lives on wavefronts in flight: five a SIMD with blocks of
    two, eight else (the compiler may form the quotients of all mantissas at once, which takes the registers of two), and
    nothing spilled."""
    out = str(tmp_path / "brute.s")
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "brute_kernels.hip"), "-o", out],
                   check=True, capture_output=True)
    found = 0
    for part in open(out).read().split("; -- Begin function ")[1:]:        # figures stand behind each kernel's end
        kernel = re.match(r"_ZN3mxq12brute_kernelILi[01]ELi(\d+)ELi[12]ELb[01]ELb1E", part)    # <type, block, format, scaled, pruned>
        if kernel:
            found += 1
            room, spilled = (int(re.search(rf"; {k}: (\d+)", part).group(1)) for k in ("Occupancy", "ScratchSize"))
            assert spilled == 0 and room >= (5 if kernel.group(1) == "2" else 8), (kernel.group(), room, spilled)
    assert found == 2 * 7 * 2 * 2
