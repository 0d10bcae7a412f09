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


def bf16_bits(v):
    return (np.asarray(v, np.float32).view(np.uint32) >> 16).astype(np.uint16)       # truncated: full mantissas stay full


def guard_blocks(block, top):
    """bf16 blocks (as fp32) on both sides of the two rules for exact squares, in wavefronts of 512 elements: {name: blocks}.
    small: every element around 2^-72 .. 2^-64, no zeros; zeros: the same with some; far: every element 64 to 4096 times the
    largest power of two up to the largest scale `top`; low: every element 64 to 4096 times some lower scale."""
    rng = np.random.default_rng(block)
    waves = 16
    shape = (waves, 512 // block, block)
    mantissa = rng.choice([-1, 1], shape) * (1 + rng.integers(0, 128, shape) / 128)
    small = mantissa * 2.0 ** (np.linspace(-72, -64, waves).round()[:, None, None] + rng.integers(-1, 2, shape))
    zeros = np.where(rng.random(shape) < 0.1, 0.0, small)
    many = 2.0 ** rng.integers(6, 13, shape)
    far = mantissa * many * 2.0 ** np.floor(np.log2(top))
    low = mantissa * many * 2.0 ** -rng.integers(4, 12, waves)[:, None, None]
    return {k: v.reshape(-1, block).astype(np.float32) for k, v in dict(small=small, zeros=zeros, far=far, low=low).items()}


@pytest.mark.parametrize("fmt", [E4M3, UE5M3])
@pytest.mark.parametrize("block", [4, 8, 16, 64])
def test_blocks_beyond_the_rules_tell_fused_sums_apart(oracle, fmt, block):
    """What a search with a rule missing would return for these blocks is not what it has to: SSEs with the odd squares of
    each lane fused, under the scales that the rule keeps from it, against separately rounded ones.  (The searches themselves
    are compared with the oracle on these blocks in test_gpu_kernel_edges.py.)"""
    def sums(v, S, fused):
        q = np.array([0, .5, 1, 1.5, 2, 3, 4, 6], np.float32)
        y = np.abs(v.astype(np.float64) / S)
        e = (np.abs(v) - q[np.abs(y[..., None] - q).argmin(-1)] * S).astype(np.float32)
        even, odd = (e[:, 0::2] * e[:, 0::2]).astype(np.float32), e[:, 1::2]
        if fused:
            first = (odd.astype(np.longdouble) ** 2 + even.astype(np.longdouble)).astype(np.float32)
        else:
            first = ((odd * odd).astype(np.float32) + even).astype(np.float32)
        return tree_sum32(first)

    top = np.float32(oracle.scale_decode(fmt, oracle.scale_max_code(fmt)))
    data = guard_blocks(block, float(top))
    assert all((bf16_bits(v).astype(np.uint32) << 16 == v.view(np.uint32)).all() for v in data.values())
    # under the scales that win: any for elements that vanish, the largest beyond the format (the lower scales of "low" never
    # win, its wavefronts only go from one kind of sum to the other)
    for name, S in (("small", np.float32(2.0 ** -6)), ("zeros", np.float32(2.0 ** -6)), ("far", top)):
        apart = int((sums(data[name], S, True) != sums(data[name], S, False)).sum())
        assert apart >= 5, (name, apart)
