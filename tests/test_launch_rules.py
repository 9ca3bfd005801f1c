"""The launch rules that are plain functions of sizes, on the CPU:
tests/sanitize/rules_driver.cpp under AddressSanitizer and
UndefinedBehaviorSanitizer (ROCm's clang as a plain host compiler, no GPU
code)."""
import os

import pytest

from test_oracle_sanitized import CLANG, ROOT, SAN, _build, _run


@pytest.mark.skipif(not os.path.exists(CLANG + "++"), reason="ROCm clang not available")
def test_launch_rules_under_sanitizers(tmp_path):
    exe = str(tmp_path / "rules_driver")
    _build([CLANG + "++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include"] + SAN +
           ["-I", os.path.join(ROOT, "include"),
            "-I", os.path.join(ROOT, "paper_1206_1187_amd", "csrc"),
            os.path.join(ROOT, "tests", "sanitize", "rules_driver.cpp"), "-o", exe])
    _run(exe, "rules driver ok")
