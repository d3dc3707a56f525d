"""Launch choices that the tuner wrote are used only with the kernels that it timed, and it times
launches in which members are active."""
import numpy as np
import pytest

import qhd_inputs
from paper_2303_01471_amd import qhd as q

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    q.load_library()


def _arch():
    import torch
    return torch.cuda.get_device_properties(0).gcnArchName.replace(" ", "_").replace(":", "_")


def _info(specs, flags, cache):
    plan = q.Plan(specs, flags=flags, tune_cache=cache)
    try:
        return plan.graph_info()["classes"][0]
    finally:
        plan.close()


def test_lines_timed_on_other_kernels_are_not_used(tmp_path):
    """A line with the timings of the separate axis passes is passed over, one without timings
    (a caller's own choice) is used; the tuner then adds a line of its own and reads it back."""
    specs = [q.InstanceSpec(shape=(128, 128), nsteps=64, dt=1e-3)] * 4
    keys = ("col_variant", "cap_row", "cap_col", "row_points")
    cache = tmp_path / "tune.txt"
    default = _info(specs, 0, None)
    old = f"qhd-tune 1 {_arch()} 128 128 4 1 512 1024 8"
    cache.write_text(old + "  # row 9.87 us, col 6.54 us\n")
    got = _info(specs, 0, str(cache))
    assert [got[k] for k in keys] == [default[k] for k in keys]
    cache.write_text(old + "\n")
    assert [_info(specs, 0, str(cache))[k] for k in keys] == [1, 512, 1024, 8]
    cache.write_text(old + "  # row 9.87 us, col 6.54 us\n")
    tuned = _info(specs, q.QHD_OPT_AUTOTUNE, str(cache))
    assert tuned["tuned"] and len(cache.read_text().splitlines()) == 2
    again = _info(specs, q.QHD_OPT_AUTOTUNE, str(cache))
    assert not again["tuned"] and [again[k] for k in keys] == [tuned[k] for k in keys]


def test_a_resident_choice_timed_on_other_kernels_is_not_used(tmp_path):
    specs = [q.InstanceSpec(shape=(64, 64), nsteps=64, dt=1e-3)] * 512
    flags = q.QHD_OPT_RESIDENT | q.QHD_OPT_AUTOTUNE
    cache = tmp_path / "tune.txt"
    old = f"qhd-resident 1 {_arch()} 64 64 512 0 0"
    cache.write_text(old + "  # 16 steps: resident 987.65 us, streaming 123.45 us\n")
    _info(specs, flags, str(cache))
    assert len([ln for ln in cache.read_text().splitlines() if ln.startswith("qhd-resident")]) == 2
    cache.write_text(old + "\n")
    assert _info(specs, flags, str(cache))["resident"] is False


def test_members_of_one_step_are_timed_at_work(tmp_path):
    """64 x 512^2 of one step each: a pass in which they are active reads and writes 24 bytes of
    each of 16.8 M points, which no memory of the card does in 20 us (20 TB/s)."""
    specs = [q.InstanceSpec(shape=(512, 512), nsteps=1, dt=1e-3)] * 64
    cache = tmp_path / "tune.txt"
    assert _info(specs, q.QHD_OPT_AUTOTUNE, str(cache))["tuned"]
    line = cache.read_text().splitlines()[-1]
    row, col = float(line.split("row ")[1].split()[0]), float(line.split("col ")[1].split()[0])
    assert row > 20.0 and col > 20.0, line


def test_members_without_steps_are_not_timed(tmp_path):
    specs = [q.InstanceSpec(shape=(64, 64), nsteps=0, dt=1e-3)] * 3
    cache = tmp_path / "tune.txt"
    assert not _info(specs, q.QHD_OPT_AUTOTUNE | q.QHD_OPT_RESIDENT, str(cache))["tuned"]
    assert not cache.exists() or cache.read_text() == ""
