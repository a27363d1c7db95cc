"""libpl.so holds a kernel for every plane pass, one-pass CG step and narrow x
tile that the host dispatches (a dispatch table that misses one fails here,
without a GPU)."""
import os
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_0911_1407_amd", "libpl.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libpl.so not built")


@pytest.fixture(scope="module")
def syms():
    return subprocess.run(["nm", "-C", LIB], capture_output=True, text=True).stdout


def test_plane_kernels(syms):
    # r2c, c2r, HVP, c2r + diagonal; in FP64 also the gradient's three and the
    # linear bias's two (the first of them for the short lengths only)
    for cls in (0, 1):
        for T, ops in (("double", (0, 1, 2, 3, 4, 5, 7, 8) + ((6,) if cls == 0 else ())), ("float", (0, 1, 2, 4))):
            for op in ops:
                assert f"plane_kernel<{T}, {op}, {cls}>" in syms, (T, op, cls)


def test_one_pass_cg_and_narrow_tiles(syms):
    from paper_0911_1407_amd import binding
    for n in binding.SUPPORTED_LENGTHS:
        variants = (0, 1, 3, 4, 5, 6) if n in (128, 192, 256, 512) else (0,)
        narrow = (2, 7) if 32 <= n <= 128 else ()
        for v in variants + narrow:
            assert f"col_kernel<double, {n}, false, 6, {v}>" in syms, (n, v)
        for T in ("double", "float"):
            for v in narrow:
                for inv, op in [("true", 0), ("false", 0), ("false", 1), ("false", 2), ("true", 3), ("false", 4),
                                ("true", 5)]:
                    assert f"col_kernel<{T}, {n}, {inv}, {op}, {v}>" in syms, (T, n, inv, op, v)
