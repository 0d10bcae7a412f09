"""What the compiler makes of the tensor abs-max (CPU only, gfx950 assembly of aux_kernels.hip).

The kernel reads the part of a large tensor that the quantise pass will find in the caches with
ordinary loads and the rest with non-temporal ones.  Written as two branches of one loop the compiler
merges the two loads and drops the hint, without a word; and a division by a run-time group size costs
a small call a tenth of its time."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_08565_amd", "csrc")


@pytest.fixture(scope="module")
def bodies(tmp_path_factory):
    from paper_2605_08565_amd.build import FLAGS
    out = str(tmp_path_factory.mktemp("asm") / "aux.s")
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    subprocess.run([hipcc, *FLAGS, "--offload-device-only", "-S", os.path.join(CSRC, "aux_kernels.hip"), "-o", out], check=True,
                   capture_output=True)
    text = open(out).read()
    found = dict(re.findall(r"^(_ZN3mxq\w*absmax\w*kernelI\w+):(.*?)s_endpgm", text, re.S | re.M))
    assert sum("absmax_kernel" in k for k in found) == 4 and sum("absmax_small_kernel" in k for k in found) == 2
    return found


def test_large_tensors_are_read_with_both_kinds_of_load(bodies):
    for name, body in bodies.items():
        loads = re.findall(r"global_load_dwordx4.*", body)
        hinted = sum(l.rstrip().endswith(" nt") for l in loads)
        if "small" in name:
            assert len(loads) >= 4 and hinted == 0, name
        else:
            assert hinted >= 4 and len(loads) - hinted >= 4, (name, loads)


def test_no_division_by_a_run_time_number(bodies):
    for name, body in bodies.items():
        assert not re.search(r"v_rcp_|v_cvt_f32_u32", body), name
