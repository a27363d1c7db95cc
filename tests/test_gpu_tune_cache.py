"""Schedule caches kept from before the FP64 CG step had one x pass: their FP64
lines are tiles for other kernels and are timed anew, not taken; the lines stay
in the file, and FP32 lines hold."""
import pytest

from paper_0911_1407_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_old_fp64_lines_are_timed_anew(tmp_path):
    from paper_0911_1407_amd import binding
    inst = synth.config_instance("plain32")
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    old = [f"{arch} 32x32x32 shell {p} 6 5 1 4 2 2 31 0.1000 0.1000" for p in ("fp64", "fp32")]
    cache = tmp_path / "tune.txt"
    cache.write_text("\n".join(old) + "\n")
    plan = binding.Plan(inst["n"], inst["box"], precision="mixed")
    plan.set_instance(inst)
    got = plan.autotune(str(cache))
    assert got["fp32"] == (6, 5, 1, 4, 2, 2, 31)
    assert got["fp64"] != (6, 5, 1, 4, 2, 2, 31)
    lines = [l for l in cache.read_text().splitlines() if not l.startswith("#")]
    assert lines[:2] == old and len(lines) == 3
    again = binding.Plan(inst["n"], inst["box"], precision="mixed")
    again.set_instance(inst)
    assert again.autotune(str(cache)) == got and len(cache.read_text().splitlines()) == 5
