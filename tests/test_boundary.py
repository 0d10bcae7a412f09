"""The C-ABI library: it loads, exports every symbol the header declares, its host helpers
agree with the oracle, and every argument error is reported before anything is launched.
No GPU needed: validation runs on the host and precedes any HIP call."""
import ctypes
import math
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def mxq():
    from paper_2605_08565_amd import mxq as M
    if not os.path.exists(M.LIB_PATH):
        from paper_2605_08565_amd.build import build_library
        build_library()
    M.lib()
    return M


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "mxq.h")).read()
    return sorted(set(re.findall(r"MXQ_API[^;(]*?\b(mxq_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol(mxq):
    names = declared_symbols()
    assert names == sorted(["mxq_quantize", "mxq_quantize_batch", "mxq_quantize_clip", "mxq_quantize_hier", "mxq_dequantize", "mxq_dequantize_hier", "mxq_tensor_absmax", "mxq_tensor_absmax_ws", "mxq_tensor_absmax_acc", "mxq_tensor_absmax_static",
                            "mxq_tensor_absmax_workspace_size", "mxq_clip_sse",
                            "mxq_histogram",
                            "mxq_tensor_scale_from_absmax", "mxq_scale_decode",
                            "mxq_num_candidates", "mxq_status_string"])
    L = ctypes.CDLL(mxq.LIB_PATH)
    for n in names:
        assert hasattr(L, n), n


def test_host_helpers_agree_with_oracle(mxq, oracle):
    for fmt in (0, 1, 2):
        assert mxq.num_candidates(fmt) == oracle.num_candidates(fmt)
        for code in range(256):
            a, b = mxq.scale_decode(fmt, code), oracle.scale_decode(fmt, code)
            assert (math.isnan(a) and math.isnan(b)) or a == b, (fmt, code)
    assert mxq.num_candidates(7) == -1
    for A in (0.0, 1.0, 250.0, 3.1e-5, 2688.0, 1e30):
        for fmt in (0, 1, 2):
            assert mxq.tensor_scale_from_absmax(A, fmt) == oracle.tensor_scale(A, fmt)
    assert mxq.tensor_scale_from_absmax(2688.0, mxq.SCALE_E4M3) == 1.0
    assert math.isnan(mxq.tensor_scale_from_absmax(1.0, 9))
    assert mxq.status_string(0) == "MXQ_OK"
    assert mxq.status_string(-3) == "MXQ_ERR_ALIGNMENT"
    assert mxq.status_string(77) == "MXQ_ERR_UNKNOWN"


def test_argument_validation_without_a_launch(mxq):
    L = mxq.lib()
    P = 0x10000  # a fake, aligned, never-dereferenced device address

    def q(x=P, rows=4, cols=64, block=16, elem=0, fmt=1, rec=0, T=1.0, codes=P, scales=P, sse=P, dt=0):
        return L.mxq_quantize(x, rows, cols, block, elem, fmt, rec, T, codes, scales, sse, dt, None)

    assert q(x=None) == mxq.ERR_INVALID_ARG
    assert q(codes=None) == mxq.ERR_INVALID_ARG
    assert q(scales=None) == mxq.ERR_INVALID_ARG
    assert q(rows=-1) == mxq.ERR_INVALID_ARG
    assert q(block=3) == mxq.ERR_INVALID_ARG
    assert q(block=256) == mxq.ERR_INVALID_ARG
    assert q(cols=72, block=16) == mxq.ERR_INVALID_ARG
    assert q(elem=1) == mxq.ERR_INVALID_ARG
    assert q(fmt=3) == mxq.ERR_INVALID_ARG
    assert q(rec=6) == mxq.ERR_INVALID_ARG and q(rec=-1) == mxq.ERR_INVALID_ARG
    assert q(dt=2) == mxq.ERR_INVALID_ARG
    for T in (0.0, -1.0, float("inf"), float("nan")):
        assert q(T=T) == mxq.ERR_INVALID_ARG
    assert q(fmt=0, rec=2) == mxq.ERR_UNSUPPORTED
    assert q(fmt=0, rec=3) == mxq.ERR_UNSUPPORTED
    assert q(fmt=0, rec=5) == mxq.ERR_UNSUPPORTED
    assert q(x=P + 2) == mxq.ERR_ALIGNMENT
    assert q(codes=P + 1) == mxq.ERR_ALIGNMENT
    assert q(scales=P + 2) == mxq.ERR_ALIGNMENT
    assert q(sse=P + 4) == mxq.ERR_ALIGNMENT
    assert q(rows=1 << 40, cols=1 << 40) == mxq.ERR_INVALID_ARG
    assert q(rows=1 << 30, cols=1 << 12) == mxq.ERR_UNSUPPORTED        # 2^42 elements: beyond the slice counters
    # empty tensors are a valid no-op, also with NULL pointers
    assert q(rows=0) == mxq.OK
    assert q(rows=0, x=None, codes=None, scales=None, sse=None) == mxq.OK
    assert q(rows=3, cols=0) == mxq.OK

    def qc(x=P, rows=4, cols=64, block=16, elem=0, fmt=1, rec=0, T=1.0, codes=P, scales=P, sse=P, clip=P, dt=0):
        return L.mxq_quantize_clip(x, rows, cols, block, elem, fmt, rec, T, codes, scales, sse, clip, dt, None)

    assert qc(x=None) == mxq.ERR_INVALID_ARG and qc(block=3) == mxq.ERR_INVALID_ARG
    assert qc(clip=P + 4) == mxq.ERR_ALIGNMENT and qc(sse=P + 8) == mxq.ERR_ALIGNMENT
    assert qc(fmt=0, rec=2) == mxq.ERR_UNSUPPORTED and qc(rows=0) == mxq.OK

    T_ = mxq._Tensor

    def qb(tensors, block=16, elem=0, fmt=1, rec=0, dt=0):
        arr = (T_ * max(len(tensors), 1))(*tensors)
        return L.mxq_quantize_batch(arr, len(tensors), block, elem, fmt, rec, dt, None)

    good = T_(P, 4, 64, P, P, P)
    assert qb([]) == mxq.OK and L.mxq_quantize_batch(None, 0, 16, 0, 1, 0, 0, None) == mxq.OK
    assert L.mxq_quantize_batch(None, 2, 16, 0, 1, 0, 0, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_quantize_batch(None, -1, 16, 0, 1, 0, 0, None) == mxq.ERR_INVALID_ARG
    assert qb([good], block=3) == mxq.ERR_INVALID_ARG and qb([good], fmt=5) == mxq.ERR_INVALID_ARG
    assert qb([good], rec=9) == mxq.ERR_INVALID_ARG and qb([good], dt=2) == mxq.ERR_INVALID_ARG
    assert qb([good], rec=4) == mxq.ERR_UNSUPPORTED and qb([good], rec=5) == mxq.ERR_UNSUPPORTED
    assert qb([good], fmt=0, rec=2) == mxq.ERR_UNSUPPORTED
    # one bad tensor anywhere in the list refuses the whole call, before any launch
    assert qb([good, T_(None, 4, 64, P, P, P)]) == mxq.ERR_INVALID_ARG
    assert qb([good, T_(P, 4, 72, P, P, P)]) == mxq.ERR_INVALID_ARG
    assert qb([good, T_(P, -4, 64, P, P, P)]) == mxq.ERR_INVALID_ARG
    assert qb([good, T_(P, 4, 64, None, P, P)]) == mxq.ERR_INVALID_ARG
    assert qb([good, T_(P + 2, 4, 64, P, P, P)]) == mxq.ERR_ALIGNMENT
    assert qb([good, T_(P, 4, 64, P, P, P + 4)]) == mxq.ERR_ALIGNMENT
    assert qb([good, T_(P, 1 << 28, 1 << 12, P, P, P)]) == mxq.ERR_UNSUPPORTED
    assert qb([T_(None, 0, 64, None, None, None), T_(P, 5, 0, P, P, P)]) == mxq.OK        # only empty tensors

    def qh(x=P, rows=4, cols=64, block=16, elem=0, fmt=1, rec=0, amax=P, t_out=P, codes=P, scales=P, sse=P, dt=0):
        return L.mxq_quantize_hier(x, rows, cols, block, elem, fmt, rec, amax, t_out, codes, scales, sse, dt, None)

    assert qh(amax=None) == mxq.ERR_INVALID_ARG
    assert qh(x=None) == mxq.ERR_INVALID_ARG and qh(block=3) == mxq.ERR_INVALID_ARG
    assert qh(fmt=0, rec=5) == mxq.ERR_UNSUPPORTED
    assert qh(amax=P + 2) == mxq.ERR_ALIGNMENT and qh(t_out=P + 1) == mxq.ERR_ALIGNMENT
    assert qh(rows=0) == mxq.OK and qh(rows=0, t_out=None) == mxq.OK

    def d(codes=P, scales=P, rows=4, cols=64, block=16, elem=0, fmt=1, T=1.0, out=P, dt=1):
        return L.mxq_dequantize(codes, scales, rows, cols, block, elem, fmt, T, out, dt, None)

    assert d(codes=None) == mxq.ERR_INVALID_ARG
    assert d(out=None) == mxq.ERR_INVALID_ARG
    assert d(block=5) == mxq.ERR_INVALID_ARG
    assert d(fmt=-1) == mxq.ERR_INVALID_ARG
    assert d(dt=3) == mxq.ERR_INVALID_ARG
    assert d(T=0.0) == mxq.ERR_INVALID_ARG
    assert d(out=P + 8) == mxq.ERR_ALIGNMENT
    assert d(rows=0) == mxq.OK

    def dh(codes=P, scales=P, rows=4, cols=64, block=16, elem=0, fmt=1, t=P, out=P, dt=1):
        return L.mxq_dequantize_hier(codes, scales, rows, cols, block, elem, fmt, t, out, dt, None)

    assert dh(t=None) == mxq.ERR_INVALID_ARG and dh(codes=None) == mxq.ERR_INVALID_ARG
    assert dh(t=P + 2) == mxq.ERR_ALIGNMENT and dh(rows=0) == mxq.OK

    def cl(x=P, scales=P, rows=4, cols=64, block=16, elem=0, fmt=1, T=1.0, out=P, dt=0):
        return L.mxq_clip_sse(x, scales, rows, cols, block, elem, fmt, T, out, dt, None)

    assert cl(x=None) == mxq.ERR_INVALID_ARG and cl(scales=None) == mxq.ERR_INVALID_ARG
    assert cl(out=None) == mxq.ERR_INVALID_ARG and cl(block=7) == mxq.ERR_INVALID_ARG
    assert cl(T=-2.0) == mxq.ERR_INVALID_ARG and cl(fmt=4) == mxq.ERR_INVALID_ARG
    assert cl(out=P + 4) == mxq.ERR_ALIGNMENT and cl(rows=0) == mxq.OK

    def hi(codes=P, scales=P, rows=4, cols=64, block=16, elem=0, eh=P, sh=P):
        return L.mxq_histogram(codes, scales, rows, cols, block, elem, eh, sh, None)

    assert hi(codes=None) == mxq.ERR_INVALID_ARG and hi(eh=None) == mxq.ERR_INVALID_ARG
    assert hi(sh=None) == mxq.ERR_INVALID_ARG and hi(cols=70) == mxq.ERR_INVALID_ARG
    assert hi(eh=P + 4) == mxq.ERR_ALIGNMENT and hi(codes=P + 2) == mxq.ERR_ALIGNMENT

    assert L.mxq_tensor_absmax(P, 4, 4, 0, None, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax(None, 4, 4, 0, P, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax(P, 4, 4, 5, P, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax(P + 4, 4, 4, 0, P, None) == mxq.ERR_ALIGNMENT

    # the allocation-free form: argument errors and the size limit come before any HIP call
    assert L.mxq_tensor_absmax_static(P, 4, 4, 0, None, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax_static(None, 4, 4, 0, P, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax_static(P, 4, 4, 3, P, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax_static(P + 4, 4, 4, 0, P, None) == mxq.ERR_ALIGNMENT
    assert L.mxq_tensor_absmax_static(P, 1 << 21, (1 << 19) + 8, 0, P, None) == mxq.ERR_UNSUPPORTED
    assert L.mxq_tensor_absmax_acc(P, 4, 4, 0, None, None, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax_acc(P, 4, 4, 0, P, P, None) == mxq.ERR_INVALID_ARG       # same word
    assert L.mxq_tensor_absmax_acc(P, 4, 4, 0, P, P + 6, None) == mxq.ERR_ALIGNMENT
    assert L.mxq_tensor_absmax_acc(None, 4, 4, 0, P, P + 4, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax_acc(None, 0, 4, 0, P, None, None) == mxq.OK                # nothing to do

    wsz = L.mxq_tensor_absmax_workspace_size()
    assert wsz == 256
    assert L.mxq_tensor_absmax_ws(P, 4, 4, 0, P, None, wsz, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax_ws(P, 4, 4, 0, P, P, wsz - 1, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax_ws(P, 4, 4, 0, P, P + 4, wsz, None) == mxq.ERR_ALIGNMENT
    assert L.mxq_tensor_absmax_ws(P, 4, 4, 0, None, P, wsz, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax_ws(None, 4, 4, 0, P, P, wsz, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax_ws(P, 4, 4, 7, P, P, wsz, None) == mxq.ERR_INVALID_ARG
    assert L.mxq_tensor_absmax_ws(P + 8, 4, 4, 1, P, P, wsz, None) == mxq.ERR_ALIGNMENT


def test_binding_fails_loudly_without_the_library(mxq, monkeypatch):
    monkeypatch.setattr(mxq, "_lib", None)
    monkeypatch.setattr(mxq, "LIB_PATH", "/nonexistent/libmxq.so")
    with pytest.raises(ImportError):
        mxq.lib()


def test_header_is_plain_c_and_links(tmp_path, mxq):
    """include/mxq.h compiles as strict C99 and a C program linked against libmxq.so can call the
    host helpers (no GPU needed)."""
    import subprocess
    src = tmp_path / "use_mxq.c"
    src.write_text('#include "mxq.h"\n'
                   '#include <stdio.h>\n'
                   'int main(void) {\n'
                   '    printf("%d %d %g %s\\n", mxq_num_candidates(MXQ_SCALE_E4M3), mxq_num_candidates(MXQ_SCALE_UE5M3),\n'
                   '           (double)mxq_scale_decode(MXQ_SCALE_E4M3, 0x7E), mxq_status_string(MXQ_ERR_ALIGNMENT));\n'
                   '    return 0;\n'
                   '}\n')
    exe = tmp_path / "use_mxq"
    libdir = os.path.dirname(mxq.LIB_PATH)
    subprocess.run(["gcc", "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror", "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe), "-L", libdir, "-lmxq", f"-Wl,-rpath,{libdir}"], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split()
    assert out == ["126", "254", "448", "MXQ_ERR_ALIGNMENT"]


def test_dequantize_takes_tensors_beyond_one_grid_in_pieces(tmp_path):
    """The launcher's own code with a recording stand-in for the runtime's kernel launch."""
    import shutil
    import subprocess
    from paper_2605_08565_amd.build import FLAGS
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    exe = str(tmp_path / "launch_pieces_check")
    subprocess.run([hipcc, *FLAGS, os.path.join(ROOT, "tests", "host", "launch_pieces_check.hip"),
                    os.path.join(ROOT, "paper_2605_08565_amd", "csrc", "aux_kernels.hip"), "-o", exe], check=True, capture_output=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(res.stdout)
    assert res.returncode == 0 and "cases=196 bad=0" in res.stdout
