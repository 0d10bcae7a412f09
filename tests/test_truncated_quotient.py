"""Element quotients by one truncated product: the arithmetic on the CPU, the kernels' rounding on the GPU."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2605_08565_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
CLANG = shutil.which("amdclang++") or "/opt/rocm/llvm/bin/clang++"


def test_decisions_of_the_truncated_quotient_are_exact(tmp_path):
    exe = str(tmp_path / "truncated_quotient_check")
    subprocess.run([CLANG, "-O2", "-std=c++17", "-ffp-contract=off", "-Wall", "-Werror",
                    os.path.join(HERE, "host", "truncated_quotient_check.cpp"), "-o", exe, "-lm"], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300).stdout
    print(out)
    lines = [l for l in out.splitlines() if "cases=" in l]
    assert [l.split()[0] for l in lines] == ["bf16_values"]
    for l in lines:
        assert int(l.split("cases=")[1].split()[0]) > 1_000_000 and int(l.split("bad=")[1]) == 0, l


def tie_blocks(oracle, fmt, block, seed):
    """bf16 blocks for every scale code: abs-max 6 S (4 S under 4-over-6's other candidate), the other elements
    on the rounding ties of S and on the bf16 values next to them, both signs."""
    rng = np.random.default_rng(seed)
    ties = np.array([.25, .75, 1.25, 1.75, 2.5, 3.5, 5.0], np.float32)
    rows = []
    for code in range(1, oracle.scale_max_code(fmt) + 1):
        s = np.float32(oracle.scale_decode(fmt, code))
        for top in (6.0, 4.0):
            v = W.f32_to_bf16_bits(rng.choice(ties, block) * s) + rng.integers(-1, 2, block).astype(np.uint16)
            v[rng.integers(block)] = W.f32_to_bf16_bits(np.float32([top]) * s)[0]
            rows.append(v | (rng.integers(0, 2, block).astype(np.uint16) << np.uint16(15)))
    return np.stack(rows).astype(np.uint16)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("block", [2, 4, 8, 16, 128])
def test_ties_of_every_scale_code(oracle, fmt, block):
    """Codes, scales and SSE are bits: no tolerance."""
    from paper_2605_08565_amd import mxq

    x = tie_blocks(oracle, fmt, block, seed=17 * block + fmt)
    gx = mxq.from_bits(x)
    for recipe in (0, 1, 2, 3):
        want = oracle.quantize(x, block, fmt, recipe)
        for got in (mxq.quantize(gx, block, fmt, recipe), mxq.quantize_batch([gx], block, fmt, recipe)[0]):
            torch.cuda.synchronize()
            for g, r in zip(got, want):
                g = g.cpu().numpy()
                assert (g.view(np.uint32) == r.view(np.uint32)).all() if g.dtype == np.float32 else (g == r).all(), (recipe, g.dtype)
