"""The native forms of the binding's calls (csrc/binding.cpp) against the Python forms, which define them."""
import ctypes
import os
import subprocess

import pytest
import torch

from paper_2605_08565_amd import mxq


def test_native_calls_are_built_and_decline_what_is_not_plain():
    """On the CPU: None before anything is done for CPU tensors, other types and active modes."""
    mxq.lib()
    assert os.path.exists(os.path.join(os.path.dirname(mxq.__file__), "_mxq_calls.so")) and mxq._calls is not None
    x = torch.zeros((4, 32), dtype=torch.bfloat16)
    u = torch.zeros((4, 16), dtype=torch.uint8)
    for v in (x, None, 3, "x", torch.nn.Parameter(x.float()), x.expand(4, 32)):
        assert mxq._calls.quantize(v, 16, 1, 0, 1.0, None, None, None, True, 0) is None
        assert mxq._calls.quantize_hier(v, 16, 1, 0, x, None, None, None, None, True, 0) is None
        assert mxq._calls.quantize_batch([v], 16, 1, 0, True, 0) is None
        assert mxq._calls.tensor_absmax(v, None) is None
        assert mxq._calls.clip_sse(v, u, 16, 1, 1.0, None, 0) is None
    assert mxq._calls.dequantize(u, u, 16, 1, 1.0, torch.float32, None, 0) is None
    assert mxq._calls.histogram(u, u, 16, 0) is None
    assert mxq._calls.quantize_batch([], 16, 1, 0, True, 0) is None


def test_native_calls_of_another_build_are_not_used(tmp_path, monkeypatch):
    """Layouts of torch and signatures of mxq.h are compiled into the module: neither may differ from what is loaded."""
    from paper_2605_08565_amd import build

    L = mxq.lib()
    assert mxq._native_calls(L) is not None and mxq.calls_abi() == build.calls_abi()
    assert mxq._native_calls(L).built_for() == (mxq.calls_abi(), ctypes.string_at(ctypes.addressof(
        ctypes.c_char.in_dll(L, "mxq_header_id"))).decode())
    assert torch.__version__ in mxq.calls_abi() and torch.version.git_version in mxq.calls_abi()
    for name, text in (("other", 'const char mxq_header_id[] = "0123456789abcdef";'), ("without", "int mxq_nothing;")):
        (tmp_path / f"{name}.c").write_text(text)
        so = str(tmp_path / f"{name}.so")
        subprocess.run(["gcc", "-shared", "-fPIC", str(tmp_path / f"{name}.c"), "-o", so], check=True)
        assert mxq._native_calls(ctypes.CDLL(so)) is None, name
    monkeypatch.setattr(mxq, "calls_abi", lambda: "cpython-310 2.9.1 0")
    assert mxq._native_calls(L) is None


@pytest.mark.parametrize("lacking", ["torch", "g++"])
def test_c_library_is_linked_without_what_the_native_calls_need(monkeypatch, lacking):
    from paper_2605_08565_amd import build

    ran = []

    def run(cmd, verbose):
        ran.append(cmd)
        if cmd[0] == lacking:
            raise RuntimeError(f"{cmd[0]} failed")

    def no_torch():
        raise ImportError("No module named 'torch'")

    monkeypatch.setattr(build, "_run", run)
    if lacking == "torch":
        monkeypatch.setattr(build, "_calls_command", no_torch)
        assert build.build_library() == build.LIB
    else:
        with pytest.raises(RuntimeError, match=r"^g\+\+ failed"):
            build.build_library()
    assert any("-shared" in c and build.LIB in c and c[0] == "hipcc" for c in ran)


def test_a_failing_tool_is_named():
    from paper_2605_08565_amd import build

    for cmd, text in ((["gcc", "-no-such-option"], "^gcc failed"), (["no-such-compiler-here"], "^no-such-compiler-here is not installed")):
        with pytest.raises(RuntimeError, match=text):
            build._run(cmd, False)


def outcome(call):
    """What a call gives: its tensors (bit patterns), or the type and text of its error."""
    def flat(r):
        if isinstance(r, torch.Tensor):
            return (tuple(r.shape), r.dtype, r.requires_grad, r.cpu().view(torch.uint8).flatten().tolist())
        return [flat(i) for i in r] if isinstance(r, (list, tuple)) else r
    try:
        r = call()
        torch.cuda.synchronize()
        return type(r), flat(r)
    except Exception as e:
        return type(e), str(e)


@pytest.mark.gpu
@pytest.mark.parametrize("where", ["default stream", "side stream", "default device set"])
def test_native_and_python_forms_agree(monkeypatch, where):
    mxq.lib()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    x = torch.randn((6, 64), generator=gen, device="cuda", dtype=torch.float32)
    xb, n = x.to(torch.bfloat16), x.numel()
    word = mxq.tensor_absmax(x)
    codes, scales, sse, _ = mxq.quantize_hier(x, 16, 1, 2, word)

    def new(dtype, size):
        return torch.full((size,), 7, dtype=dtype, device="cuda")

    calls = {
        "quantize": lambda: mxq.quantize(xb, 16, 1, 2),
        "no sse, int scale": lambda: mxq.quantize(x, 2, 2, 0, tensor_scale=2, want_sse=False),
        "buffers": lambda: mxq.quantize(xb, 4, 1, 5, 0.5, new(torch.uint8, n // 2), new(torch.uint8, n // 4), new(torch.float32, n // 4)),
        "short buffer": lambda: mxq.quantize(xb, 4, 1, 0, codes_out=new(torch.uint8, n // 2 - 1)),
        "buffer type": lambda: mxq.quantize(xb, 4, 1, 0, sse_out=new(torch.float64, n)),
        "misaligned": lambda: mxq.quantize(xb, 4, 1, 0, codes_out=new(torch.uint8, n)[1:]),
        "block 3": lambda: mxq.quantize(xb[:, :63].contiguous(), 3, 1, 0),
        "block 0": lambda: mxq.quantize(xb, 0, 1, 0),
        "block too large": lambda: mxq.quantize(xb, 128, 1, 0),
        "recipe": lambda: mxq.quantize(xb, 16, 1, 9),
        "unsupported": lambda: mxq.quantize(xb, 16, 0, 2),
        "scale": lambda: mxq.quantize(xb, 16, 1, 2, tensor_scale=float("inf")),
        "type": lambda: mxq.quantize(x.double(), 16, 1, 2),
        "strided": lambda: mxq.quantize(x.t(), 2, 1, 2),
        "three dimensions": lambda: mxq.quantize(x.view(2, 3, 64), 16, 1, 2),
        "empty": lambda: mxq.quantize(xb[:0], 16, 1, 2),
        "parameter": lambda: mxq.quantize(torch.nn.Parameter(x), 16, 1, 2),
        "hier": lambda: mxq.quantize_hier(xb, 8, 2, 3, word),
        "hier empty": lambda: mxq.quantize_hier(xb[:0], 8, 2, 3, word),
        "hier buffers": lambda: mxq.quantize_hier(x, 8, 1, 0, word, new(torch.float32, 1), want_sse=False),
        "hier word": lambda: mxq.quantize_hier(x, 8, 1, 0, x.double()),
        "batch": lambda: mxq.quantize_batch([xb, xb[:2], xb[:0]], 32, 1, 2),
        "batch types": lambda: mxq.quantize_batch([xb, x], 32, 1, 2),
        "batch generator": lambda: mxq.quantize_batch((t for t in (x, x)), 32, 1, 2, want_sse=False),
        "batch recipe": lambda: mxq.quantize_batch([xb], 32, 1, 4),
        "absmax": lambda: mxq.tensor_absmax(xb),
        "absmax 3-d, buffer": lambda: mxq.tensor_absmax(x.view(2, 3, 64), out=new(torch.float32, 1)),
        "absmax empty": lambda: mxq.tensor_absmax(x[:0]),
        "absmax type": lambda: mxq.tensor_absmax(x.half()),
        "dequantize": lambda: mxq.dequantize(codes, scales, 16, 1, 0.25, torch.bfloat16),
        "dequantize hier": lambda: mxq.dequantize(codes, scales, 16, 1, word),
        "dequantize out": lambda: mxq.dequantize(codes, scales, 16, 1, out=new(torch.bfloat16, n)),
        "dequantize type": lambda: mxq.dequantize(codes, scales, 16, 1, out_dtype=torch.float16),
        "dequantize short": lambda: mxq.dequantize(codes, scales[:5], 16, 1),
        "clip": lambda: mxq.clip_sse(x, scales, 16, 1),
        "clip out": lambda: mxq.clip_sse(xb, scales, 16, 1, 0.5, out=new(torch.float32, n // 16)),
        "histogram": lambda: mxq.histogram(codes, scales, 16),
        "histogram block": lambda: mxq.histogram(codes, scales, 24),
    }
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())

    def everything():
        if where == "side stream":
            with torch.cuda.stream(side):
                return {k: outcome(c) for k, c in calls.items()}
        if where == "default device set":                               # a mode: the native forms decline
            with torch.device("cuda"):
                return {k: outcome(c) for k, c in calls.items()}
        return {k: outcome(c) for k, c in calls.items()}

    native = everything()
    monkeypatch.setattr(mxq, "_calls", None)
    python = everything()
    for k in calls:
        assert native[k] == python[k], k
    assert native["quantize"][0] is tuple and native["misaligned"][0] is mxq.MxqError and native["strided"][0] is ValueError


def native_calls(x, word, codes, scales):
    """One plain call of each native form, outputs allocated there: name -> (call, the Python call it stands for)."""
    c = mxq._calls
    return {
        "quantize": (lambda: c.quantize(x, 16, 1, 2, 1.0, None, None, None, True, 0), lambda: mxq.quantize(x, 16, 1, 2)),
        "quantize_hier": (lambda: c.quantize_hier(x, 16, 1, 2, word, None, None, None, None, True, 0),
                          lambda: mxq.quantize_hier(x, 16, 1, 2, word)),
        "quantize_batch": (lambda: c.quantize_batch([x, x], 32, 2, 0, True, 0), lambda: mxq.quantize_batch([x, x], 32, 2, 0)),
        "tensor_absmax": (lambda: c.tensor_absmax(x, None), lambda: mxq.tensor_absmax(x)),
        "dequantize": (lambda: c.dequantize(codes, scales, 16, 1, 1.0, torch.bfloat16, None, 0),
                       lambda: mxq.dequantize(codes, scales, 16, 1, 1.0, torch.bfloat16)),
        "clip_sse": (lambda: c.clip_sse(x, scales, 16, 1, 1.0, None, 0), lambda: mxq.clip_sse(x, scales, 16, 1)),
        "histogram": (lambda: c.histogram(codes, scales, 16, 0), lambda: mxq.histogram(codes, scales, 16)),
    }


@pytest.mark.gpu
def test_native_forms_take_plain_calls_and_decline_under_modes():
    from torch.overrides import TorchFunctionMode

    mxq.lib()
    x = torch.randn((64, 1024), device="cuda").to(torch.bfloat16)
    word = mxq.tensor_absmax(x)
    codes, scales, _ = mxq.quantize(x, 16, 1, 2)
    calls = native_calls(x, word, codes, scales)
    for name, (native, _) in calls.items():
        assert native() is not None, name
    with TorchFunctionMode():
        for name, (native, _) in calls.items():
            assert native() is None, name
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_native_forms_in_a_captured_graph(monkeypatch):
    """Captured, a call is recorded only if it goes to the current stream; replayed on new contents it must give what the
    Python form gives on them, with eager work and synchronisation in between."""
    mxq.lib()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    x = torch.randn((64, 1024), generator=gen, device="cuda").to(torch.bfloat16)
    word = mxq.tensor_absmax(x)
    codes, scales, _ = mxq.quantize(x, 16, 1, 2)
    calls = native_calls(x, word, codes, scales)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                                       # warm-up outside capture
        for native, _ in calls.values():
            native()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = {name: native() for name, (native, _) in calls.items()}
    assert all(r is not None for r in captured.values())
    with monkeypatch.context() as m:
        m.setattr(mxq, "_calls", None)

        def flat(r):
            return [r] if isinstance(r, torch.Tensor) else [t for i in r for t in flat(i)]

        for seed in range(4):
            gen.manual_seed(100 + seed)
            x.copy_(torch.randn(x.shape, generator=gen, device="cuda") * (seed + 1))
            word.copy_(x.abs().max().reshape(1))
            for t, new in zip((codes, scales), mxq.quantize(x, 16, 1, 3)):
                t.copy_(new)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for name, (_, python) in calls.items():
                for g, w in zip(flat(captured[name]), flat(python())):
                    assert torch.equal(g.view(torch.uint8), w.view(torch.uint8)), (seed, name)


def test_new_outputs_go_past_the_dispatcher_only_where_nothing_watches_it():
    mxq.lib()
    direct = mxq._calls.new_outputs_direct
    assert direct()
    with torch.inference_mode():
        assert direct()
    with torch.no_grad():
        assert direct()
    torch.use_deterministic_algorithms(True)                   # has new memory filled
    try:
        assert not direct()
    finally:
        torch.use_deterministic_algorithms(False)
    seen = []
    torch.func.vmap(lambda y: seen.append(direct()) or y + 1)(torch.zeros(3))
    torch.func.grad(lambda y: seen.append(direct()) or y.sum())(torch.zeros(3))
    torch.jit.trace(lambda y: seen.append(direct()) or y + 1, torch.zeros(3), check_trace=False)
    assert len(seen) >= 3 and not any(seen)
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU]):
        assert not direct()
    with torch.autograd.profiler.profile(use_device=None):
        assert not direct()
    assert direct()


@pytest.mark.gpu
def test_a_profiler_sees_the_outputs_of_the_native_calls_made():
    x = torch.randn((64, 64), device="cuda")
    mxq.quantize(x, 16, 1, 0)
    torch.cuda.synchronize()
    counts = []
    for call in (lambda: mxq.quantize(x, 16, 1, 0), lambda: mxq.quantize(x, 16, 1, 0, want_sse=False)):
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CPU]) as p:
            call()
        counts.append(sum(e.count for e in p.key_averages() if e.key == "aten::empty"))
    assert counts == [3, 2]


@pytest.mark.gpu
def test_new_outputs_of_the_native_calls_are_those_of_torch_empty():
    """The same kind of tensor in inference mode, on the inputs' device and in the caching allocator's books, and the same
    results where new memory is filled or a transform is active (which way they are allocated there is the test of
    new_outputs_direct)."""
    x = torch.randn((64, 64), device="cuda")
    want = mxq.quantize(x, 16, 1, 0)

    def same(got):
        torch.cuda.synchronize()
        for g, w in zip(got, want):
            assert g.dtype == w.dtype and g.shape == w.shape and g.stride() == w.stride() and g.device == w.device
            assert torch.equal(g, w) and not g.requires_grad and g.is_contiguous()

    before = torch.cuda.memory_allocated()
    got = mxq.quantize(x, 16, 1, 0)
    assert torch.cuda.memory_allocated() - before == sum(-(-t.numel() * t.element_size() // 512) * 512 for t in got)
    same(got)
    with torch.inference_mode():
        got = mxq.quantize(x, 16, 1, 0)
        assert all(t.is_inference() for t in got)
    same(got)
    assert not any(t.is_inference() for t in mxq.quantize(x, 16, 1, 0))
    torch.use_deterministic_algorithms(True)
    try:
        same(mxq.quantize(x, 16, 1, 0))
    finally:
        torch.use_deterministic_algorithms(False)
    seen = []

    def f(y):
        seen.append(mxq.quantize(x, 16, 1, 0))
        return y + 1

    torch.func.vmap(f)(torch.zeros(3, device="cuda"))
    same(seen[0])
    with torch.no_grad():
        same(mxq.quantize(x, 16, 1, 0))
