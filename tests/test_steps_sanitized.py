"""The FP64 steps of the default kernels, chained, on the CPU:
tests/sanitize/steps_driver.cpp against the oracle under AddressSanitizer and
UndefinedBehaviorSanitizer (ROCm's clang as a plain host compiler, no GPU
code)."""
import os

import pytest

from test_oracle_sanitized import CLANG, ROOT, SAN, _build, _run


@pytest.mark.skipif(not os.path.exists(CLANG + "++"), reason="ROCm clang not available")
def test_steps_chained_under_sanitizers(tmp_path):
    obj = str(tmp_path / "nn_oracle.o")
    exe = str(tmp_path / "steps_driver")
    _build([CLANG, "-std=c11", "-Wno-unknown-pragmas"] + SAN +
           ["-I", os.path.join(ROOT, "oracle"), "-c",
            os.path.join(ROOT, "oracle", "nn_oracle.c"), "-o", obj])
    _build([CLANG + "++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include"] + SAN +
           ["-I", os.path.join(ROOT, "include"),
            "-I", os.path.join(ROOT, "paper_1206_1187_amd", "csrc"),
            "-I", os.path.join(ROOT, "oracle"),
            os.path.join(ROOT, "tests", "sanitize", "steps_driver.cpp"), obj, "-o", exe])
    _run(exe, "steps driver ok")
