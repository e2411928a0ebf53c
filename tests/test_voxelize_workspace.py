"""Where the voxelizer keeps its slot counter."""
from tests.test_fixed_point import run_program


def test_the_counters_line_is_its_own(tmp_path):
    run_program(tmp_path, "vox_workspace_case.cpp", "emu.cpp")
