"""GPU results at the sizes and values where a kernel's own branches meet: window edges of the
pruned scale search, tile and tail edges.  Everything is compared bit for bit with the oracle."""
import numpy as np
import pytest
import torch

from paper_2605_08565_amd import workloads as W
from test_pruning_bounds import bf16_bits, guard_blocks

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mxq():
    from paper_2605_08565_amd import mxq as M
    assert torch.cuda.is_available(), "these tests need the GPU"
    M.lib()
    return M


def same(gpu, ref):
    torch.cuda.synchronize()
    for g, r, name in zip(gpu, ref, ("codes", "scales", "sse")):
        g = g.cpu().numpy()
        assert (g.view(np.uint32) == r.view(np.uint32)).all() if name == "sse" else (g == r).all(), name


def window_edge_blocks(oracle, fmt, block, seed):
    """fp32 blocks whose abs-max sits on, just below and just above 3.5, 4, 5, 6 and 1/4 times a scale,
    the other elements on grid points and rounding ties of that scale, for codes over the whole range."""
    rng = np.random.default_rng(seed)
    top = oracle.scale_max_code(fmt)
    codes = sorted(set(range(1, 34)) | {top - 9, top - 8, top - 1, top} | set(rng.integers(34, top, 24).tolist()))
    grid = np.array([0, .25, .5, .75, 1, 1.25, 1.5, 1.75, 2, 2.5, 3, 3.5], np.float32)
    rows = []
    for c in codes:
        s = np.float32(oracle.scale_decode(fmt, c))
        for f in (3.5, 4.0, 5.0, 6.0, 0.25, 40.0):
            a = np.float32(f) * s
            for amax in (a, np.nextafter(a, np.float32(0)), np.nextafter(a, np.float32(np.inf))):
                v = rng.choice(grid, block) * s if rng.random() < 0.5 else rng.random(block).astype(np.float32) * amax
                v = np.minimum(v.astype(np.float32), amax) * rng.choice([-1, 1], block)
                v[rng.integers(block)] = amax
                rows.append(v.astype(np.float32))
    return np.stack(rows)


@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("block", [2, 4, 8, 16, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_pruned_search_window_edges(oracle, mxq, fmt, block, dtype):
    x = window_edge_blocks(oracle, fmt, block, seed=31 * block + fmt)
    if dtype == "bf16":
        x = W.f32_to_bf16_bits(x)
    print(f"[edges] pruned fmt={fmt} b={block} {dtype} blocks={x.shape[0]}", flush=True)
    for T in (1.0, 0.7):
        ref = oracle.quantize(x, block, fmt, 4, tensor_scale=T)
        same(mxq.quantize(mxq.from_bits(x), block, fmt, mxq.RECIPE_BRUTE_PRUNED, tensor_scale=T), ref)


@pytest.mark.parametrize("T", [1.0, 0.7])
@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("block", [2, 4, 8, 16])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_pruned_search_in_wavefronts_of_normal_scales(oracle, mxq, fmt, block, dtype, T):
    """The unrolled way up runs only where EVERY block of a wavefront (512 elements) starts at a code from
    16 to top - 7, so whole wavefronts of such blocks are made: all codes of that range, its two ends in
    every wavefront, the abs-max on and beside 3.5, 4, 5 and 6 times a scale.  Behind them wavefronts
    with a single block one code too low and one too high, which send it the general way."""
    rng = np.random.default_rng(100 * block + 10 * fmt + (dtype == "bf16"))
    top, per_wave = oracle.scale_max_code(fmt), 512 // block
    grid = np.array([0, .25, .5, .75, 1, 1.25, 1.5, 1.75, 2, 2.5, 3, 3.5], np.float32)

    def make(codes, factors):
        """One block per (code, factor, neighbour) and the codes that the abs-max rule gives them."""
        c, f, d = (a.ravel() for a in np.meshgrid(codes, factors, (-1, 0, 1), indexing="ij"))
        s = np.array([oracle.scale_decode(fmt, int(i)) for i in c], np.float32) * np.float32(T)
        step = 1 if dtype == "f32" else 1 << 16
        amax = (((s * f.astype(np.float32)).view(np.uint32) // step + d.astype(np.uint32)) * step).astype(np.uint32).view(np.float32)
        v = np.where(rng.random((len(c), 1)) < 0.5, rng.choice(grid, (len(c), block)) * s[:, None], rng.random((len(c), block)) * amax[:, None])
        v = np.minimum(v, amax[:, None]) * rng.choice([-1, 1], (len(c), block))
        v[np.arange(len(c)), rng.integers(block, size=len(c))] = amax
        x = v.astype(np.float32)
        x = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
        return x, oracle.quantize(x, block, fmt, 0, tensor_scale=T)[1][:, 0].astype(int)

    x, start = make(np.arange(16, top + 1), (3.5, 4.0, 5.0, 6.0))
    x, start = x[(start >= 16) & (start <= top - 7)], start[(start >= 16) & (start <= top - 7)]
    ends = np.concatenate([x[start == 16][:1], x[start == top - 7][:1]])
    out, out_start = make([15, top - 6], (6.0,))
    low, high = out[out_start < 16][:1], out[out_start > top - 7][:1]
    x = x[rng.permutation(len(x))]
    body = per_wave - 3
    waves = [np.concatenate([ends, x[i:i + body], x[:1]]) for i in range(0, len(x) - body, body)]
    waves[-2][-1], waves[-1][-1] = low[0], high[0]
    x = np.concatenate(waves)
    start = oracle.quantize(x, block, fmt, 0, tensor_scale=T)[1][:, 0].astype(int).reshape(len(waves), per_wave)
    inside = ((start >= 16) & (start <= top - 7))
    assert inside.all(axis=1).sum() == len(waves) - 2 >= 2 and (inside.sum(axis=1)[-2:] == per_wave - 1).all()
    assert (start[:-2].min(axis=1) == 16).all() and (start[:-2].max(axis=1) == top - 7).all()
    print(f"[edges] fast wavefronts fmt={fmt} b={block} {dtype} T={T} wavefronts={len(waves)}", flush=True)
    same(mxq.quantize(mxq.from_bits(x), block, fmt, mxq.RECIPE_BRUTE_PRUNED, tensor_scale=T),
         oracle.quantize(x, block, fmt, 4, tensor_scale=T))


@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("block", [2, 4, 8, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_pruned_search_beyond_the_format(oracle, mxq, fmt, block, dtype):
    """Blocks whose abs-max lies above 6 times the largest scale, alone in their wavefront and beside
    ordinary ones, up to magnitudes at which the codes no longer differ and at which every SSE overflows;
    NaN and infinity, whose codes are not specified but whose scale byte and SSE are the full search's."""
    rng = np.random.default_rng(block + 7 * fmt)
    top = 6 * oracle.scale_decode(fmt, oracle.scale_max_code(fmt))
    n = 4 * 512 // block                                    # four wavefronts of each kind
    rows = []
    for e in (0, 0.1, 1, 3, 8, 16, 24, 26, 28, 40):
        x = rng.standard_normal((n, block)) * top * 2.0 ** e
        rows += [x, np.where(rng.random((n, 1)) < 0.1, x, rng.standard_normal((n, block)) * 0.02),
                 np.sign(x) * top * 2.0 ** e * (1 + 0.05 * rng.random((n, block)))]
    x = np.concatenate(rows).astype(np.float32)
    x = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    print(f"[edges] beyond fmt={fmt} b={block} {dtype} blocks={x.shape[0]}", flush=True)
    same(mxq.quantize(mxq.from_bits(x), block, fmt, mxq.RECIPE_BRUTE_PRUNED), oracle.quantize(x, block, fmt, 4))
    x = (rng.standard_normal((n, block)) * 0.02).astype(np.float32)
    for i, bad in enumerate((np.nan, np.inf, -np.inf, 3e38, 1.8e19, 1.9e19)):
        x[7 * i::61, i % block] = bad
    g = mxq.from_bits(W.f32_to_bf16_bits(x) if dtype == "bf16" else x)
    full, pruned = mxq.quantize(g, block, fmt, mxq.RECIPE_BRUTE), mxq.quantize(g, block, fmt, mxq.RECIPE_BRUTE_PRUNED)
    torch.cuda.synchronize()
    assert torch.equal(full[1], pruned[1]) and torch.equal(full[2], pruned[2])
    ok = torch.isfinite(g.float()).all(dim=1)
    assert torch.equal(full[0][ok], pruned[0][ok])


@pytest.mark.parametrize("block", [2, 4])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_ragged_tail_beside_full_slices(oracle, mxq, block, dtype):
    """n = 8 * 256 * k + r: the tail of r < 8 elements is handled inside the main launch, alone (k = 0),
    behind exactly full slices and behind a part-filled one; single calls, batches, all outputs."""
    rng = np.random.default_rng(5 * block)
    xs = []
    for n in [n0 + r for n0 in (0, 8, 2048, 6 * 2048, 6 * 2048 + 1000) for r in (block, 8 - block)]:
        x = (rng.standard_normal((1, n)) * 0.05).astype(np.float32)
        xs.append(W.f32_to_bf16_bits(x) if dtype == "bf16" else x)
    for x in xs:
        print(f"[edges] tail b={block} {dtype} n={x.size}", flush=True)
        g = mxq.from_bits(x)
        for fmt, rec, T in [(0, 0, 1.0), (1, 2, 0.7), (2, 3, 1.0), (1, 4, 1.0), (2, 5, 0.7)]:
            ref = oracle.quantize(x, block, fmt, min(rec, 4), tensor_scale=T)
            same(mxq.quantize(g, block, fmt, rec, tensor_scale=T), ref)
            clip = torch.full(ref[2].shape, -1.0, device="cuda")
            same(mxq.quantize(g, block, fmt, rec, tensor_scale=T, clip_sse_out=clip), ref)
            want = oracle.clip_sse(x, ref[1], block, fmt, tensor_scale=T)
            assert (clip.cpu().numpy().view(np.uint32) == want.view(np.uint32)).all()
        amax = mxq.tensor_absmax(g)
        *out, t = mxq.quantize_hier(g, block, 1, 2, amax)
        same(out, oracle.quantize(x, block, 1, 2, tensor_scale=float(t.cpu()[0])))
    for out, x in zip(mxq.quantize_batch([mxq.from_bits(x) for x in xs], block, 1, 3), xs):
        same(out, oracle.quantize(x, block, 1, 3))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tensor_absmax_around_the_one_workgroup_limit(oracle, mxq, dtype):
    """One workgroup up to 160 KiB, two launches beyond; the maximum first, last and in between; all forms."""
    limit = (160 << 10) // (4 if dtype == "f32" else 2)
    ws, words = mxq.absmax_workspace(), torch.full((3,), 7.0, device="cuda")
    for n in (1, 7, 8, 9, 8 * 1024, 4 * 8 * 1024 + 3, limit - 8, limit, limit + 1, limit + 8):
        for at in {0, n // 2, n - 1}:
            x = np.linspace(-1, 1, n, dtype=np.float32).reshape(1, n)
            x[0, at] = -3.0
            x = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
            print(f"[edges] absmax {dtype} n={n} at={at}", flush=True)
            g = mxq.from_bits(x)
            mxq.tensor_absmax(g, out=words[0:1])
            mxq.tensor_absmax(g, out=words[1:2], workspace=ws)
            mxq.tensor_absmax_static(g, words[2:3])
            assert words.cpu().tolist() == [3.0] * 3
    assert int(ws.sum()) == 0


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tensor_absmax_at_group_edges(mxq, dtype):
    """Eight workgroups share a group of 512 KiB slice by slice, 32 groups are in flight: the maximum in the
    first and last element of slices, groups and the tensor, sizes around one, two and 32 groups."""
    size = 4 if dtype == "f32" else 2
    per = (512 << 10) // size
    word = torch.empty(1, device="cuda")
    ws = mxq.absmax_workspace()
    for n in (per // 2 + 5, per - 8, per, per + 8, 2 * per + 2048 * 3 + 1, 32 * per, 33 * per + 13):
        x = torch.zeros((1, n), dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
        at = {0, 2047, 2048, 8 * 2048 - 1, 8 * 2048, per // 2, per - 1, per, n // 8 * 8 - 1, n - 1}
        print(f"[edges] absmax groups {dtype} n={n}", flush=True)
        for value, i in enumerate(sorted(i for i in at if i < n), start=1):
            x[0, i] = -float(value)                        # the latest one is the largest
            assert float(mxq.tensor_absmax(x, out=word).cpu()[0]) == value
            assert float(mxq.tensor_absmax(x, workspace=ws).cpu()[0]) == value
            assert float(mxq.tensor_absmax_acc(x, torch.zeros(1, device="cuda")).cpu()[0]) == value


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tensor_absmax_with_few_tiles_and_at_the_change_of_loads(mxq, dtype):
    """One workgroup per tile of 64 KiB up to eight tiles, whole teams beyond, two tiles a workgroup with
    tickets beyond 64 of them; and both sides of the 64 MiB where the kind of load changes."""
    size = 4 if dtype == "f32" else 2
    tile, keep = (64 << 10) // size, (64 << 20) // size
    word, ws = torch.empty(1, device="cuda"), mxq.absmax_workspace()
    sizes = [1, 8, tile - 8, tile, tile + 1, 3 * tile + 9, 7 * tile, 8 * tile, 8 * tile + 1, 9 * tile + 8, 64 * tile, 65 * tile, 129 * tile + 3]
    for n in sizes + [keep, keep + 8, keep + 8 * tile + 1, keep + 300 * tile]:
        x = torch.zeros((1, n), dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
        at = {0, 255, tile - 1, tile, 5 * tile + 77, 8 * tile - 1, 8 * tile, keep - 1, keep, n // 2, n // 8 * 8 - 1, n - 1}
        print(f"[edges] absmax tiles {dtype} n={n}", flush=True)
        for value, i in enumerate(sorted(i for i in at if 0 <= i < n), start=1):
            x[0, i] = -float(value)                        # the latest one is the largest
            assert float(mxq.tensor_absmax(x, out=word).cpu()[0]) == value
            assert float(mxq.tensor_absmax(x, workspace=ws).cpu()[0]) == value
            assert float(mxq.tensor_absmax_static(x, word).cpu()[0]) == value
            assert float(mxq.tensor_absmax_acc(x, torch.zeros(1, device="cuda")).cpu()[0]) == value
    assert int(ws.sum()) == 0


@pytest.mark.parametrize("block", [2, 4, 8, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_dequantize_at_tile_edges(oracle, mxq, block, dtype):
    """One chunk per lane up to 2048 workgroups, four (or three) beyond: remainders of a chunk, of a workgroup's tile and
    the line between the two, T by value and from device memory."""
    rng = np.random.default_rng(block)
    per = 8 if dtype == "bf16" else 4
    line = 2048 * 256 * per
    out_dtype = torch.bfloat16 if dtype == "bf16" else torch.float32
    beyond = [line + k * 256 * per + d for k in (3, 4) for d in (-block, block)]
    if dtype == "bf16" and block < 8:                      # three chunks per lane beyond 2048 workgroups of four
        beyond += [4 * line + d for d in (-block, 0, block, 3 * 256 * per - block, 3 * 256 * per + block)]
    for n in (block, 256 * per - block, 256 * per + block, 1024 * per + 8, line - block, line, line + block, *beyond):
        n = n // block * block
        if n == 0:
            continue
        codes = rng.integers(0, 256, (1, n // 2), dtype=np.uint8)
        scales = rng.integers(0, 0x7F, (1, n // block), dtype=np.uint8)
        print(f"[edges] dequantize {dtype} b={block} n={n}", flush=True)
        want = oracle.dequantize(codes, scales, block, 1, 0.75)
        c, s = torch.from_numpy(codes).cuda(), torch.from_numpy(scales).cuda()
        for t in (0.75, torch.full((1,), 0.75, device="cuda")):
            out = torch.full((1, n + 8), 7.0, dtype=out_dtype, device="cuda")     # nothing beyond n may change
            mxq.dequantize(c, s, block, 1, t, out_dtype, out=out)
            got = out.float().cpu().numpy()
            ref = want if dtype == "f32" else torch.from_numpy(want).to(torch.bfloat16).float().numpy()
            assert (got[:, :n] == ref).all() and (got[:, n:] == 7.0).all()


@pytest.mark.parametrize("block", [2, 4, 8, 16, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_quantize_where_a_workgroup_takes_three_slices(oracle, mxq, block, dtype):
    """From 16384 slices of 2048 elements on: one slice below the line, tiles of three that end full, one and two slices
    short, a part-filled last slice, a ragged tail.  Whole tensors against the quantisation of their pieces (below the
    line, where a workgroup loops), which no tile boundary shares, and the last elements against the oracle."""
    rng = np.random.default_rng(block)
    per, line = 2048, 16384
    period = (rng.standard_normal(block * 40009) * 0.05).astype(np.float32)
    big = torch.from_numpy(np.resize(period, (line + 3) * per)).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16)
    ends = [(line - 1) * per, line * per, (line + 1) * per, (line + 1) * per + 1000 // block * block]
    if block < 8:
        ends.append((line + 2) * per + 6 // block * block)
    for n in ends:
        x = big[:n].reshape(1, n)
        for fmt, rec, T, want in [(1, 2, 1.0, True), (2, 1, 1.0, False), (0, 0, 1.0, True), (1, 0, 0.7, True)]:
            print(f"[edges] large b={block} {dtype} n={n} fmt={fmt} recipe={rec} T={T}", flush=True)
            for got in (mxq.quantize(x, block, fmt, rec, tensor_scale=T, want_sse=want),
                        *(mxq.quantize_batch([x], block, fmt, rec, want_sse=want) if T == 1.0 else ())):
                cut = n // 3 // block * block
                pieces = [mxq.quantize(x[:, i:j].clone(), block, fmt, rec, tensor_scale=T, want_sse=want)
                          for i, j in ((0, cut), (cut, 2 * cut), (2 * cut, n))]
                assert (got[2] is not None) == want
                for g, *p in zip(got if want else got[:2], *pieces):
                    assert torch.equal(g.view(torch.uint8), torch.cat(p, 1).view(torch.uint8))
                end = x[:, n - 5 * per - n % per:].contiguous()
                end = end.cpu().numpy() if dtype == "f32" else end.view(torch.int16).cpu().numpy().view(np.uint16)
                ref = oracle.quantize(end, block, fmt, rec, tensor_scale=T)
                same([g[:, -r.shape[1]:].contiguous() for g, r in zip(got, ref) if g is not None], ref)


@pytest.mark.parametrize("block", [2, 4, 16, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_batch_where_a_workgroup_takes_three_slices_of_one_tensor(oracle, mxq, block, dtype):
    """Eleven tensors: the first eight that are not empty, more than 16384 slices together, in one launch of workgroups that
    take three slices of a tensor and end, the rest in one of workgroups that loop.  A large tensor among the eight, one and two
    slices more than a multiple of three, part-filled last slices, a tensor of one block, an empty one, ragged tails (b = 2, 4);
    with and without SSEs.  Small tensors whole and the large one's end against the oracle, the whole of
    it against single calls on its pieces."""
    rng = np.random.default_rng(block)
    per, tail = 2048, 6 // block * block
    sizes = [per, 2 * per + 8 * block + tail, block, 16390 * per + 1000 // block * block + tail, 0, 4 * per + tail, 5 * per, 3 * per + 128 + tail,
             7 * per + tail, block, 10 * per]
    period = (rng.standard_normal(block * 40009) * 0.05).astype(np.float32)
    kind = torch.float32 if dtype == "f32" else torch.bfloat16
    xs = [torch.from_numpy(np.resize(np.roll(period, 977 * i), n)).cuda().to(kind).reshape(1, n) for i, n in enumerate(sizes)]
    assert all(n % block == 0 for n in sizes) and sum(-(-n // per) for n in sizes[:8]) >= 16384
    for fmt, rec, want in ((1, 2, True), (2, 1, False), (0, 0, True)):
        print(f"[edges] large batch b={block} {dtype} fmt={fmt} recipe={rec} sse={want}", flush=True)
        outs = mxq.quantize_batch(xs, block, fmt, rec, want_sse=want)
        for i, (x, got) in enumerate(zip(xs, outs)):
            n = sizes[i]
            assert (got[2] is not None) == want and got[0].numel() == n // 2 and got[1].numel() == n // block
            if n == 0:
                continue
            if n > 16384 * per:
                cut = n // 3 // block * block
                pieces = [mxq.quantize(x[:, a:b].clone(), block, fmt, rec, want_sse=want) for a, b in ((0, cut), (cut, 2 * cut), (2 * cut, n))]
                for g, *p in zip(got if want else got[:2], *pieces):
                    assert torch.equal(g.view(torch.uint8), torch.cat(p, 1).view(torch.uint8)), i
            end = x[:, max(0, n - 6 * per - n % per):].contiguous()
            end = end.cpu().numpy() if dtype == "f32" else end.view(torch.int16).cpu().numpy().view(np.uint16)
            ref = oracle.quantize(end, block, fmt, rec)
            same([g[:, -r.shape[1]:].contiguous() for g, r in zip(got, ref) if g is not None], ref)


@pytest.mark.parametrize("T", [1.0, 0.7])
@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("block", [2, 4, 8, 16, 64])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_pruned_search_in_a_window_of_eight_codes(oracle, mxq, fmt, block, dtype, T):
    """Wavefronts (512 elements) whose blocks all start at code 17 or above and lie within the format try eight codes
    mantissa by mantissa: both ends of that range, the last codes of the format, where the window moves down, abs-max values
    on and beside 3.5, 6 and 6.5 times a scale; beside them wavefronts with one block outside it; elements that are zero,
    nearly vanish or tie."""
    rng = np.random.default_rng(1000 * block + 10 * fmt + (dtype == "bf16"))
    top, per_wave = oracle.scale_max_code(fmt), 512 // block
    value = lambda c: np.float32(oracle.scale_decode(fmt, int(c)))
    waves = []
    for kind in range(24):
        codes = rng.integers(17, top + 1, per_wave)
        codes[:4] = (18, top, top - 6, top - 7) if per_wave >= 4 else codes[:4]
        s = np.array([value(c) for c in codes], np.float32)
        f = rng.choice([3.5, 5.0, 6.0, 6.0, 6.49], per_wave).astype(np.float32)
        f[codes < 30] = np.maximum(f[codes < 30], 6.0)                   # 6 S at least: the start is not below 17
        amax = f * s
        v = rng.choice([0.25, 0.75, 1.25, 1.75, 2.5, 3.5, 5.0, 1.0, 1.5, 3.0], (per_wave, block)) * s[:, None]
        v = np.where(rng.random((per_wave, 1)) < 0.5, v, rng.random((per_wave, block)) * amax[:, None])
        v = np.minimum(v, amax[:, None])
        if kind % 4 == 1:
            v[rng.random(v.shape) < 0.2] = 0.0
        if kind % 4 == 2:
            v[rng.random(v.shape) < 0.2] = 2.0 ** rng.integers(-74, -60)
        v = v * rng.choice([-1, 1], v.shape)
        v[np.arange(per_wave), rng.integers(block, size=per_wave)] = amax
        if kind >= 20:                                                    # one block outside the range
            v[rng.integers(per_wave)] = (value(16) * 5.5, value(top) * 6.6, 0.0, value(3))[kind - 20]
        waves.append(v.astype(np.float32) * np.float32(T))
    x = np.concatenate(waves)
    x = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    print(f"[edges] window fmt={fmt} b={block} {dtype} T={T}", flush=True)
    same(mxq.quantize(mxq.from_bits(x), block, fmt, mxq.RECIPE_BRUTE_PRUNED, tensor_scale=T),
         oracle.quantize(x, block, fmt, 4, tensor_scale=T))


@pytest.mark.parametrize("T", [1.0, 0.7])
@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("block", [2, 16, 32, 64, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_pruned_search_goes_on_down_behind_its_window(oracle, mxq, fmt, block, dtype, T):
    """Blocks that the window takes and whose best code may lie more than eight below it: values spread evenly over their
    range (b = 128: some 15 steps down), and two-valued blocks, in wavefronts of their own, mixed with ordinary blocks and
    with a NaN among them (for which all codes are tried again)."""
    rng = np.random.default_rng(7 * block + fmt)
    per_wave = 512 // block
    even = rng.uniform(-1, 1, (12 * per_wave, block)) * 2.0 ** rng.integers(-1, 6, (12 * per_wave, 1))
    two = np.where(rng.random((6 * per_wave, block)) < 0.5, 1.0, rng.uniform(0.05, 0.6, (6 * per_wave, 1))) * rng.choice([-1, 1], (6 * per_wave, block))
    mixed = rng.standard_normal((6 * per_wave, block))
    mixed[::3] = rng.uniform(-1, 1, mixed[::3].shape)
    x = (np.concatenate([even, two, mixed]) * T).astype(np.float32)
    x[-per_wave * 2, 0] = np.nan
    x = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    print(f"[edges] behind the window fmt={fmt} b={block} {dtype} T={T}", flush=True)
    got = mxq.quantize(mxq.from_bits(x), block, fmt, mxq.RECIPE_BRUTE_PRUNED, tensor_scale=T)
    ref = oracle.quantize(x, block, fmt, 4, tensor_scale=T)
    rows = np.arange(x.shape[0]) != x.shape[0] - per_wave * 2
    assert (got[1].cpu().numpy() == ref[1]).all()                          # the block of the NaN too: code 1
    same([g.cpu()[torch.from_numpy(rows)].cuda() for g in got], [r[rows] for r in ref])


@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("block", [4, 8, 32])
def test_search_where_squares_are_exact_and_where_not(oracle, mxq, fmt, block):
    """bf16 wavefronts on both sides of what lets a search sum exact squares: elements on and beside 128 times every power of
    two of the scales, on and beside 2^-67, zeros; both searches."""
    rng = np.random.default_rng(block + fmt)
    rows = 512 // block
    waves = []
    for e in range(-20, 20):
        for m in (1.0, 0.99609375, 1.9921875):
            v = rng.standard_normal((rows, block)) * 2.0 ** (e - 9)
            v[0, 0] = m * 2.0 ** e
            if e % 4 == 1:
                v[-1, -1] = 2.0 ** rng.integers(-70, -64) * m
            if e % 4 == 2:
                v[-1, -1] = 0.0
            waves.append(v)
    x = W.f32_to_bf16_bits(np.concatenate(waves).astype(np.float32))
    print(f"[edges] squares fmt={fmt} b={block}", flush=True)
    ref = oracle.quantize(x, block, fmt, 4)
    for recipe in (mxq.RECIPE_BRUTE, mxq.RECIPE_BRUTE_PRUNED):
        same(mxq.quantize(mxq.from_bits(x), block, fmt, recipe), ref)


@pytest.mark.parametrize("fmt", [1, 2])
@pytest.mark.parametrize("block", [4, 8, 16, 64])
def test_search_beyond_the_rules_for_exact_squares(oracle, mxq, fmt, block):
    """Blocks whose SSEs come out otherwise where a rule is missing (shown in test_pruning_bounds.py), each kind in wavefronts
    of its own: both searches against the oracle."""
    top = float(oracle.scale_decode(fmt, oracle.scale_max_code(fmt)))
    for name, v in guard_blocks(block, top).items():
        x = bf16_bits(v)
        ref = oracle.quantize(x, block, fmt, 4)
        for recipe in (mxq.RECIPE_BRUTE, mxq.RECIPE_BRUTE_PRUNED):
            print(f"[edges] rules fmt={fmt} b={block} {name} recipe={recipe}", flush=True)
            same(mxq.quantize(mxq.from_bits(x), block, fmt, recipe), ref)


@pytest.mark.parametrize("block", [2, 4, 16, 128])
def test_histogram_at_the_edges_of_its_workgroups(oracle, mxq, block):
    """A workgroup counts 64 KiB of codes or 32 KiB of scales: one for each array (which stores its counts), one for one and
    two for the other, several; vectors that begin up to three dwords into the arrays, bytes outside them."""
    rng = np.random.default_rng(block)
    kib = 2048                                             # elements in a KiB of codes
    sizes = {block, 8, 32, 40, kib, 64 * kib - 8, 64 * kib, 64 * kib + 8, 128 * kib, 128 * kib + 8, 200 * kib + 24}
    sizes |= {(32 << 10) * block + d for d in (-8, 0, 8)} if block <= 16 else set()
    for n in sorted(max(block, n // block * block) for n in sizes):
        codes = rng.integers(0, 256, n // 2, dtype=np.uint8)
        scales = (rng.integers(0, 256, n // block) if n % 3 else rng.integers(40, 44, n // block)).astype(np.uint8)
        want = [np.bincount((np.stack([codes, codes >> 4]) & 7).ravel(), minlength=8), np.bincount(scales, minlength=256)]
        for off in (0, 4, 12):
            print(f"[edges] histogram b={block} n={n} offset={off}", flush=True)
            c = torch.zeros(n // 2 + 16, dtype=torch.uint8, device="cuda")[off:off + n // 2]
            s = torch.zeros(n // block + 16, dtype=torch.uint8, device="cuda")[off:off + n // block]
            c.copy_(torch.from_numpy(codes)); s.copy_(torch.from_numpy(scales))
            got = mxq.histogram(c.reshape(1, -1), s.reshape(1, -1), block)
            assert all((g.cpu().numpy() == w).all() for g, w in zip(got, want))


@pytest.mark.parametrize("block", [2, 4, 8, 32, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_clip_sse_at_tile_edges(oracle, mxq, block, dtype):
    """A loop over chunks of 256 lanes below 16384 of them, three at once from there on: part-filled last chunks, ragged tails;
    small tensors and the ends of large ones against the oracle, large ones against their pieces."""
    rng = np.random.default_rng(block)
    line = 16384 * 2048
    period = (rng.standard_normal(block * 40009) * 0.05).astype(np.float32)
    x = torch.from_numpy(np.resize(period, line + 4 * 2048)).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16)
    last = 6 // block * block
    for n in (block, 2048, 2048 + 8 * block + last, 2048 * 2048 + 2048 + last, line - 2048, line, line + 2048 + last, line + 3 * 2048 - block):
        n = n // block * block
        print(f"[edges] clip b={block} {dtype} n={n}", flush=True)
        v = x[:n].reshape(1, n)
        for fmt, T in ((1, 1.0), (0, 0.7)):
            scales = torch.from_numpy(np.resize(rng.integers(0x10 if fmt else 0x70, 0x38 if fmt else 0x7C, 997), n // block).astype(np.uint8)).cuda().reshape(1, -1)
            got = mxq.clip_sse(v, scales, block, fmt, tensor_scale=T)
            end = min(n, 4 * 2048 + n % 2048)
            bits = v[:, n - end:].contiguous()
            bits = bits.cpu().numpy() if dtype == "f32" else bits.view(torch.int16).cpu().numpy().view(np.uint16)
            ref = oracle.clip_sse(bits, scales[:, (n - end) // block:].cpu().numpy(), block, fmt, tensor_scale=T)
            assert (got[:, (n - end) // block:].cpu().numpy().view(np.uint32) == ref.view(np.uint32)).all()
            if n >= line - 2048:
                cut = n // 3 // (4 * block) * (4 * block)
                pieces = [mxq.clip_sse(v[:, i:j].clone(), scales[:, i // block:j // block].clone(), block, fmt, tensor_scale=T)
                          for i, j in ((0, cut), (cut, 2 * cut), (2 * cut, n))]
                assert torch.equal(got.view(torch.int32), torch.cat(pieces, 1).view(torch.int32))
