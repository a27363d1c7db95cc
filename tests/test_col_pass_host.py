"""The x passes of the CG on the CPU: tests/host_kernels/col_pass_check.cpp
compiles the kernels themselves for the host, one workgroup's lanes as fibers,
and runs them where the order of waves or the range of the values matters."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_0911_1407_amd", "csrc")
# (the kernels use Clang's vector types and non-temporal builtins)
CLANG = shutil.which("clang++") or shutil.which("clang++", path="/opt/rocm/lib/llvm/bin")


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    if CLANG is None:
        pytest.skip("needs clang++")
    exe = str(tmp_path_factory.mktemp("host") / "col_pass_check")
    r = subprocess.run([CLANG, "-O1", "-std=c++17", "-I" + os.path.join(HERE, "host_kernels"), "-I" + CSRC,
                        os.path.join(HERE, "host_kernels", "col_pass_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    return r.stdout.splitlines()


def test_a_workgroup_decides_the_end_of_a_solve_as_one(lines):
    # the done flag set between the readings of a workgroup's waves, in both
    # orders: the vectors of the finished solve stay as they were
    ends = [l for l in lines if l.startswith("end ")]
    assert len(ends) == 8 and all(l.endswith("ok=1") for l in ends), "\n".join(lines)


def test_the_start_pass_sums_squares_in_64_bits(lines):
    starts = [l for l in lines if l.startswith("start ")]
    assert len(starts) == 5 and all(l.endswith("ok=1") for l in starts), "\n".join(lines)
