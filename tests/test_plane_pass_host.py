"""The plane passes on the CPU: tests/host_kernels/plane_check.cpp compiles the
kernels themselves for the host, one workgroup's lanes as fibers, and compares
them with the transforms written out as sums; a second build runs them under the
address and undefined-behaviour sanitizers."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_0911_1407_amd", "csrc")
CLANG = shutil.which("clang++") or shutil.which("clang++", path="/opt/rocm/lib/llvm/bin")


@pytest.mark.parametrize("flags", [["-O2"], ["-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"]],
                         ids=["plain", "sanitizers"])
def test_plane_passes_match_the_transforms_written_out(tmp_path, flags):
    if CLANG is None:
        pytest.skip("needs clang++")
    exe = str(tmp_path / "plane_check")
    r = subprocess.run([CLANG, "-std=c++17", *flags, "-I" + os.path.join(HERE, "host_kernels"), "-I" + CSRC,
                        os.path.join(HERE, "host_kernels", "plane_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    if r.returncode != 0 and ("asan" in r.stderr or "ubsan" in r.stderr):
        pytest.skip("sanitizer runtimes not installed: " + r.stderr[-300:])
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    lines = r.stdout.splitlines()
    assert r.returncode == 0 and len(lines) == 43 and all(l.endswith("ok=1") for l in lines), (r.stdout + r.stderr)[-4000:]
