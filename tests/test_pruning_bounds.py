"""The two lower bounds that let the pruned scale search skip codes on its way down, checked on the CPU
against the oracle's own block SSE (pinned fp32 arithmetic) for every scale code of many blocks.

  one element   while 6 S < amax the abs-max element saturates, and fl(fl(amax - 6 S)^2) is in the SSE:
                once that exceeds the best SSE found so far, the walk stops;
  all elements  the tree sum of fl(fl(|v_i| - 6 S)^2) over the saturated elements: the floor below which
                a long walk does not go.

Both must be lower bounds of the SSE under S and must not fall as S falls, so that they rule out every
lower code as well; and the lowest code of minimal SSE must survive them whatever the best SSE so far
is.  (The bound of the way up is in test_search_walk.py.)"""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = shutil.which("amdclang++") or "/opt/rocm/llvm/bin/clang++"

E4M3, UE5M3 = 1, 2


def tree_sum32(s):
    s = np.asarray(s, np.float32)
    while s.shape[-1] > 1:
        s = (s[..., 0::2] + s[..., 1::2]).astype(np.float32)
    return s[..., 0]


def blocks(kind, b, n, rng, top):
    if kind == "student":
        return (rng.standard_t(4, size=(n, b)) * 0.02).astype(np.float32)
    if kind == "normal_small":
        return (rng.standard_normal((n, b)) * 0.002).astype(np.float32)
    if kind == "outlier":
        x = rng.standard_normal((n, b)).astype(np.float32)
        x[:, 0] *= 50.0
        return x
    if kind == "flat":
        return (np.sign(rng.standard_normal((n, b))) * (1.0 + 0.05 * rng.random((n, b)))).astype(np.float32)
    if kind == "beyond":                                 # abs-max above 6 times the largest scale, up to where codes stop mattering
        return (rng.standard_normal((n, b)) * top * 2.0 ** rng.uniform(2, 40, (n, 1))).astype(np.float32)
    raise ValueError(kind)


@pytest.mark.parametrize("fmt", [E4M3, UE5M3])
@pytest.mark.parametrize("b", [4, 16])
@pytest.mark.parametrize("kind", ["student", "normal_small", "outlier", "flat", "beyond"])
def test_bounds_of_the_way_down_hold_for_every_code(oracle, fmt, b, kind):
    rng = np.random.default_rng(1000 * fmt + 10 * b + len(kind))
    max_code = oracle.scale_max_code(fmt)
    scale = np.array([oracle.scale_decode(fmt, c) for c in range(1, max_code + 1)], np.float32)
    ruled_out = 0
    for v in blocks(kind, b, 24, rng, 6.0 * float(scale[-1])):
        sse = np.array([oracle.block_sse(v, fmt, c)[1] for c in range(1, max_code + 1)], np.float32)
        over = np.maximum(np.abs(v)[None, :] - (np.float32(6.0) * scale)[:, None], np.float32(0)).astype(np.float32)
        every = tree_sum32((over * over).astype(np.float32))
        one = over.max(axis=1)
        one = (one * one).astype(np.float32)
        assert (every <= sse).all() and (one <= every).all()
        assert (np.diff(every) <= 0).all() and (np.diff(one) <= 0).all()             # ascending codes
        winner = int(np.argmin(sse))                                                 # lowest code of minimal SSE
        start = max(int(oracle.quantize(v.reshape(1, b), b, fmt, 0)[1][0, 0]), 1) - 1
        for best in (sse[start], sse[winner]):
            assert not (every[winner] > best)
            ruled_out += int((every[:start] > best).sum())
    assert ruled_out > 0 or kind == "normal_small"       # the bounds do bite


def test_squares_of_residuals_are_exact_below_512_scales():
    """A bf16 value v with |v| < 512 S leaves, under every E2M1 value q that is nearest to v / S, a residual v - q S of at
    most 12 significant bits: all 128 mantissas, all scale mantissas (four bits and the shorter ones of sub-normal codes),
    all distances of the exponents, in integers.  Beyond 512 S 13 bits occur."""
    grid = (0, 1, 2, 3, 4, 6, 8, 12)                                       # 2 q

    def most_bits(v, s):                                                   # v and s in units of 2^-24
        y2, nearest = 2 * v / s, []
        for g in grid:
            nearest.append((abs(y2 - g), g))
        best = min(nearest)[0]
        r = [abs(2 * v - g * s) for d, g in nearest if d == best]          # both sides of a tie
        return max((x // (x & -x)).bit_length() if x else 0 for x in r)

    beyond = 0
    for s_mant in list(range(8, 16)) + [1, 2, 3, 4, 5, 6, 7]:
        s = s_mant << 21                                                   # 2^24 .. for 8 .. 15
        for shift in range(-16, 13):
            for mant in range(128, 256):
                v = (mant << 17) << shift if shift >= 0 else (mant << 17) >> -shift
                if shift < 0 and (mant << 17) & ((1 << -shift) - 1):
                    continue
                if v < 512 * s:
                    assert most_bits(v, s) <= 12, (s_mant, shift, mant)
                else:
                    beyond = max(beyond, most_bits(v, s))
    assert beyond > 12


def test_fused_sums_of_squares_where_the_rules_allow_them(tmp_path):
    """The kernels' own rules (mxq_arith.hpp) over every bf16 magnitude and scale code: a zero passes them, the sums of what
    passes have the bits of separate roundings, and on either side beyond them they do not all."""
    if "fma" not in open("/proc/cpuinfo").read():
        pytest.skip("host CPU has no FMA instruction")
    exe = str(tmp_path / "squares_check")
    subprocess.run([CLANG, "-O2", "-std=c++17", "-ffp-contract=off", "-mfma", "-Wall", "-Werror",
                    os.path.join(HERE, "host", "squares_check.cpp"), "-o", exe, "-lm"], check=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(res.stdout)
    rows = {l.split()[0]: [int(t.split("=")[1]) for t in l.split()[1:]] for l in res.stdout.splitlines()}
    assert res.returncode == 0 and len(rows) == 8
    assert rows["zeros"] == [2, 0] and rows["edge"] == [3, 0]
    for fmt in ("e4m3", "ue5m3"):
        assert rows[fmt + "_inside"][0] > 1_000_000 and rows[fmt + "_inside"][1] == 0
        assert rows[fmt + "_too_small"][1] > 1000 and rows[fmt + "_too_large"][1] > 1000
