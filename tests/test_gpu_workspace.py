"""What a plan asks its caller for: six FP64 spectral vectors, five real fields
and the per-mode 1/lambda table, in a mixed plan four FP32 spectral vectors, two
FP32 fields and the FP32 table; the rest (shell tables, twiddles, partial sums,
and a batch's work lists) is less than half a spectral vector on these grids.
Solvers share the fields that are idle while they run."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def vectors(n, mixed):
    N, Nh = n[0] * n[1] * n[2], n[0] * n[1] * (n[2] // 2 + 1)
    fp64 = 6 * 16 * Nh + 5 * 8 * N + 8 * Nh
    return fp64 + (4 * 8 * Nh + 2 * 4 * N + 4 * Nh if mixed else 0), 16 * Nh


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("n", [(64, 64, 64), (96, 96, 256), (128, 128, 128)])
def test_plan_workspace(n, mixed):
    from paper_0911_1407_amd import binding
    h, ws = binding.pl_plan_create(n, tuple(float(v) for v in n), binding.PL_MIXED if mixed else binding.PL_FP64)
    binding.pl_plan_destroy(h)
    need, spectral = vectors(n, mixed)
    assert need <= ws <= need + spectral // 2, (ws, need)


@pytest.mark.parametrize("mixed", [False, True])
def test_batch_workspace(mixed):
    from paper_0911_1407_amd import binding
    ns = [(64, 64, 64), (96, 96, 96), (128, 64, 96)]
    h, ws = binding.pl_batch_create(ns, [tuple(float(v) for v in n) for n in ns],
                                    binding.PL_MIXED if mixed else binding.PL_FP64)
    binding.pl_batch_destroy(h)
    need = sum(vectors(n, mixed)[0] for n in ns)
    assert need <= ws <= need + sum(vectors(n, mixed)[1] for n in ns) // 2, (ws, need)
