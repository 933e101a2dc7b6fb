"""The weight packing of the bf16 kernels (csrc/kern_igemm_bf16.h), as compiled for the GPU: a pair's two weights are requested
together, before either is waited for, and each weight is read once whatever the number of planes."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FORMS = [(1, "false"), (2, "false"), (3, "false"), (3, "true")]


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_both_loads_of_a_pair_are_in_flight_together(tmp_path):
    src = tmp_path / "pack.hip"
    src.write_text('#include <hip/hip_runtime.h>\n#include "kern_igemm_bf16.h"\nnamespace mcn {\n' + "".join(
        "template __global__ void igemm_pack_weights_bf16_kernel<%d, %s>(const float *, unsigned *, PackParams);\n" % f for f in FORMS) + "}\n")
    out = tmp_path / "pack.s"
    subprocess.check_call([HIPCC, "-S", "--cuda-device-only", "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature",
                           "-Xclang", "-packed-fp32-ops", "-w", "-I", os.path.join(ROOT, "paper_1412_4564_amd", "csrc"), "-o", str(out), str(src)])
    bodies = dict(re.findall(r"^(_ZN3mcn30igemm_pack_weights_bf16_kernel\w+):(.*?)s_endpgm", out.read_text(), re.M | re.S))
    assert len(bodies) == len(FORMS), list(bodies)
    for name, body in bodies.items():
        code = re.findall(r"^\s+(global_load_dword|global_store_dword|s_waitcnt vmcnt)", body, re.M)
        planes = int(re.search(r"ILi(\d)E", name).group(1))
        assert code[:2] == ["global_load_dword"] * 2 and code.count("global_load_dword") == 2, (name, code)
        assert code.count("global_store_dword") == planes, (name, code)
