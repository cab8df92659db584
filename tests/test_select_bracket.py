"""The selection's sample bracket (select_plan.hpp), built for the CPU: at large
budgets and long contexts its candidates fit their list, so that no unit of
independent scores falls through to the slow general path (results alone, which
are the same on every path, cannot show that)."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SAN = os.path.join(ROOT, "tests", "sanitize")
CSRC = os.path.join(ROOT, "paper_2609_08131_amd", "csrc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no ROCm toolchain")
def test_candidates_fit(tmp_path):
    exe = str(tmp_path / "select_bracket")
    r = subprocess.run([HIPCC, "-O2", "-std=c++17", "--offload-host-only", "-x", "hip", f"-I{CSRC}",
                        os.path.join(SAN, "select_bracket.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "brackets ok" in r.stdout, r.stdout + r.stderr
