"""The greedy launcher's host code built for the CPU against stand-ins for the
runtime (tests/sanitize/greedy_launch.cpp): calls of different lengths, which may
come from several host threads, never change the LDS limit of a kernel function
that they share. No GPU is used."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CLANG = "/opt/rocm/llvm/bin/clang++"
SAN = os.path.join(ROOT, "tests", "sanitize")
CSRC = os.path.join(ROOT, "paper_2609_08131_amd", "csrc")


@pytest.mark.skipif(not (os.path.exists(HIPCC) and os.path.exists(CLANG)), reason="no ROCm toolchain")
def test_lds_limit_is_the_same_for_every_batch(tmp_path):
    flags = ["-O1", "-std=c++17", "--offload-host-only", "-x", "hip",
             f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}"]
    objs = []
    for src in (os.path.join(CSRC, "k_greedy.hip"), os.path.join(SAN, "greedy_launch.cpp")):
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        r = subprocess.run([HIPCC, *flags, "-c", src, "-o", obj], capture_output=True, text=True)
        assert r.returncode == 0, r.stdout + r.stderr
        objs.append(obj)
    exe = str(tmp_path / "greedy_launch")
    # no device code is built: its address, which only the registration stand-in sees, is 0
    r = subprocess.run([CLANG, "-no-pie", *objs, "-Wl,--unresolved-symbols=ignore-all", "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "greedy launch ok" in r.stdout, r.stdout + r.stderr
