"""Host-side rules of the biased schemes (csrc/cfd_biased_plan.h) on the CPU, under the sanitizers:
the LDS tile the host allots covers every index the selected kernel instance uses, and the queues
that its work is dealt to balance."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_biased_plan_rules(tmp_path):
    exe = str(tmp_path / "biased_plan_selftest")
    for cmd in (["g++", "-std=gnu++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-g", "-O1",
                 "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                 "-I" + os.path.join(ROOT, "paper_2302_14858_amd", "csrc"),
                 os.path.join(ROOT, "tests", "sanitize", "biased_plan_selftest.cpp"), "-o", exe], [exe]):
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, r.stdout + r.stderr
    assert "OK (0 failures)" in r.stdout, r.stdout
