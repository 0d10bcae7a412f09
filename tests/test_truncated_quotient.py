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
    if "fma" not in open("/proc/cpuinfo").read():
        pytest.skip("host CPU has no FMA instruction")
    exe = str(tmp_path / "truncated_quotient_check")
    subprocess.run([CLANG, "-O2", "-std=c++17", "-ffp-contract=off", "-mfma", "-Wall", "-Werror",
                    os.path.join(HERE, "host", "truncated_quotient_check.cpp"), "-o", exe, "-lm"], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=300).stdout
    print(out)
    lines = [l for l in out.splitlines() if "cases=" in l]
    assert [l.split()[0] for l in lines] == ["bf16_values", "tensor_scales_of_bf16_absmax", "tensor_scales", "powers_of_two"]
    for l in lines:
        assert int(l.split("cases=")[1].split()[0]) > 1_000_000 and int(l.split("bad=")[1].split()[0]) == 0, l
    assert int(lines[1].split("refused=")[1]) == 2 * 4 * 4              # four of 128, both formats, four exponents
    assert int(lines[2].split("refused=")[1]) < 300                     # of 3007


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


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("block", [2, 4, 8, 16, 128])
def test_tensor_scales_of_large_bf16_tensors(oracle, fmt, block):
    """Four tiles and a rest for every workgroup (n not a multiple of 8 for b = 2 and 4), so that the kernel for
    scaled bf16 runs: an abs-max whose tensor scale takes reciprocals from above (249), one whose scale is refused (228), an ordinary one, scales
    by value inside and outside the range that is tried, and one with an all-ones mantissa.  Rows of every tile against the
    oracle, the whole tensor against its pieces, which are small enough for the general kernel.  Bits: no tolerance."""
    from paper_2605_08565_amd import mxq

    rng = np.random.default_rng(7 * block + fmt)
    cols = 16 * block + (block if block < 8 else 0)
    rows = (4 * 2048 * 2048 + 5 * 2048) // cols + 1
    x = (rng.standard_normal(rows * cols, dtype=np.float32) * np.repeat(np.float32([1.0, 40.0]), [rows * cols // 2, rows * cols - rows * cols // 2]))
    x = W.f32_to_bf16_bits(np.clip(x, -200, 200)).reshape(rows, cols)
    # rows that are compared with the oracle: around the planted abs-max, and those of whole slices of 2048 elements, which
    # the 2048 workgroups take in turn, from every tile
    per_slice = -(-2048 // cols) + 1
    slices = [2048 * k + j for k in range(5) for j in ((0, 700, 2047) if k < 4 else (0, 4))]
    part = np.unique(np.r_[0:20, rows // 2 - 20:rows // 2 + 20, rows - 20:rows,
                           np.concatenate([np.arange(per_slice) + s * 2048 // cols for s in slices]).clip(max=rows - 1)])
    covered = {s for s in slices if set(range(s * 2048 // cols, -(-(s + 1) * 2048 // cols))) <= set(part.tolist())}
    assert covered == set(slices)
    cuts = list(range(0, rows, 2048 * 2000 // cols // 16 * 16)) + [rows]             # of at most 2000 slices
    for top in (249.0, 228.0, 225.0):
        x[rows // 2, 3] = W.f32_to_bf16_bits(np.float32([-top]))[0]
        gx = mxq.from_bits(x)
        T = oracle.tensor_scale(top, fmt)
        runs = [(T, mxq.quantize_hier(gx, block, fmt, rec, mxq.tensor_absmax(gx)), rec) for rec in (1, 2)]
        if top == 225.0:
            for t in (T, 3.0e-7, 0.7, float(np.float32(1.99999988)), 2.0 ** -61):
                runs.append((t, mxq.quantize(gx, block, fmt, 2, tensor_scale=t), 2))
            for a in (1.9999999e-15, 3.0e36):                           # T = 2^-61 and less, and beyond 2^60, derived on the device
                word = torch.full((1,), a, dtype=torch.float32, device="cuda")
                runs.append((oracle.tensor_scale(a, fmt), mxq.quantize_hier(gx, block, fmt, 2, word), 2))
        torch.cuda.synchronize()
        for t, got, rec in runs:
            want = oracle.quantize(np.ascontiguousarray(x[part]), block, fmt, rec, tensor_scale=t)
            for g, r in zip(got[:3], want):
                g = g.cpu().numpy()[part]
                assert (g.view(np.uint32) == r.view(np.uint32)).all() if g.dtype == np.float32 else (g == r).all(), (top, t, rec, g.dtype)
            pieces = [mxq.quantize(gx[a:b], block, fmt, rec, tensor_scale=t) for a, b in zip(cuts, cuts[1:])]
            for i in range(3):
                assert torch.equal(got[i].view(torch.uint8), torch.cat([p[i] for p in pieces]).view(torch.uint8)), (top, t, rec, i)
            if len(got) == 4:
                assert float(got[3].cpu()[0]) == t


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("block", [4, 16, 64])
def test_infinities_of_large_bf16_tensors(fmt, block):
    """An infinite element gives in the kernel for scaled bf16 what it gives in the general one, which small tensors
    take: under the tensor scale 1 that an infinite abs-max leads to, and under scales by value beyond 2^+-20.  (Within,
    the general kernel's refined division makes a NaN of it: the next test.)"""
    from paper_2605_08565_amd import mxq

    cols, rows = 4096, 4 * 2048 * 2048 // 4096 + 3
    gen = torch.Generator(device="cuda")
    gen.manual_seed(block)
    x = torch.randn((rows, cols), generator=gen, device="cuda").to(torch.bfloat16)
    special = (0, rows // 2, rows - 1)
    for i in special:
        x[i, 5 + i % 7::97] = float("inf")
        x[i, 40::131] = -float("inf")
    small = torch.stack([x[i] for i in special])
    word = mxq.tensor_absmax(x)
    assert float(word) == float("inf")
    for call in (lambda t: mxq.quantize_hier(t, block, fmt, 2, word), lambda t: mxq.quantize_hier(t, block, fmt, 0, word),
                 *(lambda t, T=T: mxq.quantize(t, block, fmt, 2, tensor_scale=T) for T in (2.0 ** -30, 2.0 ** 21, 3.0e-9))):
        got, want = call(x), call(small)
        for g, w in zip(got[:3], want[:3]):
            g = torch.stack([g[i] for i in special])
            assert torch.equal(g.view(torch.uint8), w.view(torch.uint8))


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("block", [2, 4, 8, 16, 128])
def test_elements_that_are_not_finite_do_not_depend_on_the_size(fmt, block):
    """Infinities, NaNs of both signs and finite elements whose quotient by T overflows: the same bytes in a tensor of many
    tiles (kernel for scaled bf16) as in one of three rows (general kernel).  A row is eight wavefronts in both.  (An SSE
    that is a NaN need only be one: which of two NaNs their sum is depends on the order of its operands, which the
    compiler is free to choose.)"""
    from paper_2605_08565_amd import mxq

    cols, rows = 4096, 4 * 2048 * 2048 // 4096 + 3
    gen = torch.Generator(device="cuda")
    gen.manual_seed(block)
    x = torch.randn((rows, cols), generator=gen, device="cuda").to(torch.bfloat16)
    bits = x.view(torch.int16)
    special = (0, rows // 2, rows - 1)
    for i, row in enumerate(special):                                   # one kind alone in a wavefront, and together
        for j, value in enumerate((0x7F80, 0xFF80, 0x7FC0, 0xFFC1, 0x7F7F, 0xFF7F)):
            at = bits[row, 512 * j + i:512 * (j + 1):97]
            at.copy_(torch.full_like(at, value - 65536 if value > 32767 else value))
            bits[row, 3584 + 61 * j + i] = value - 65536 if value > 32767 else value
    small = torch.stack([x[i] for i in special])
    calls = [lambda t, a=a, rec=rec: mxq.quantize_hier(t, block, fmt, rec, torch.full((1,), a, device="cuda"))
             for rec in (1, 2) for a in (249.0, 0.0, 225.0, 672.0, 1.0e-2, 3.0e-15, 1.0e20, float("inf"))]
    calls += [lambda t, T=T, rec=rec: mxq.quantize(t, block, fmt, rec, tensor_scale=T)
              for rec in (0, 3) for T in (0.7, 0.25, 2.0 ** -20, 3.0e-7, 2.0 ** 21)]
    for i, call in enumerate(calls):
        got, want = call(x), call(small)
        for g, w in zip(got[:3], want[:3]):
            g = torch.stack([g[j] for j in special])
            same = g == w
            if g.dtype == torch.float32:
                same = (g.view(torch.int32) == w.view(torch.int32)) | (g.isnan() & w.isnan())
            assert bool(same.all()), (i, g.dtype, int((~same).sum()))
