"""The step vector-Jacobian product in the form that the kernels run, without the
phi component (tests/sanitize/adjoint_nophi_check.cpp), compiled for the host:
plain, under ASan/UBSan and MemorySanitizer, and with automatic variables
initialised to a pattern and to zero; every build prints the same line."""
import os
import re
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2202_00086_amd", "csrc")
SRC = os.path.join(HERE, "sanitize", "adjoint_nophi_check.cpp")
HIPCC = "/opt/rocm/bin/hipcc"
CLANG = "/opt/rocm/llvm/bin/clang++"

pytestmark = pytest.mark.slow


def test_step_vjp_without_phi(tmp_path):
    lines = {}
    for mode, flags in (("plain", []), ("asan_ubsan", ["-Xarch_host", "-fsanitize=address", "-Xarch_host",
                                                       "-fsanitize=undefined"]), ("msan", None),
                        ("pattern", ["-ftrivial-auto-var-init=pattern"]), ("zero", ["-ftrivial-auto-var-init=zero"])):
        exe = str(tmp_path / mode)
        if flags is None:
            # no HIP runtime linked: MemorySanitizer needs every linked library instrumented
            cmd = [CLANG, "-x", "hip", "--offload-host-only", "-nogpulib", "-no-hip-rt", "-std=c++17", "-g", "-O1",
                   "-Xarch_host", "-fsanitize=memory", "-I/opt/rocm/include", "-D__HIP_PLATFORM_AMD__"]
        else:
            cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-g", "-O1", *flags]
        subprocess.run(cmd + ["-w", "-I", CSRC, "-o", exe, SRC], check=True, capture_output=True)
        p = subprocess.run([exe], capture_output=True, text=True, timeout=300,
                           env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0"))
        assert p.returncode == 0 and "Sanitizer" not in p.stderr and "runtime error" not in p.stderr, p.stderr[-3000:]
        lines[mode] = p.stdout.strip()
    assert len(set(lines.values())) == 1, lines
    v = {k: float(x) for k, x in re.findall(r"(\w+) ([-+0-9.e]+)", lines["plain"])}
    # the dropped terms are products with zero: rounding at most
    assert v["form"] < 1e-13 and v["fd"] < 1e-6 and v["split"] < 1e-13 and v["r_end"] < 2.5, v
