"""Where the voxelizer keeps its slot counter, and its slots."""
import numpy as np
import pytest

from oracle import vct_voxelize as vx
from tests.hostemu.driver import run_voxelize
from tests.test_fixed_point import run_program
from tests.test_host_emulation import checked  # noqa: F401  (the build fixture)


def test_the_counters_line_is_its_own(tmp_path):
    run_program(tmp_path, "vox_workspace_case.cpp", "emu.cpp")


# 4^3 voxels and so 64 slots: 63 bounding-box pixels and their bits just fit, 64 take slots
# from the counter; 17 and 48 leave words partly used
@pytest.mark.parametrize("surface", [False, True])
@pytest.mark.parametrize("pixels", [17, 48, 63, 64, 80])
def test_slots_by_pixel_up_to_the_last(checked, tmp_path, pixels, surface):  # noqa: F811
    n = 4
    faces, single = divmod(min(pixels, 64), 16) if pixels <= 64 else (5, 0)
    tris = []
    for k in range(faces):      # half of a layer: a box of 16 pixels
        z = (k + 0.4) / n % 1.0
        tris.append([(0, 0, z), (1, 0, z), (1, 1, z)] if k % 2 else [(0, 0, z), (0, 1, z), (1, 1, z)])
    for k in range(single):     # around one pixel's centre
        x, y, z = ((k % 4) + 0.5) / n, (k // 4 + 0.5) / n, 0.9
        tris.append([(x - 0.05, y - 0.05, z), (x + 0.08, y - 0.05, z), (x - 0.05, y + 0.08, z)])
    tris = np.array(tris, np.float32)
    cols = np.random.default_rng(1).uniform(0.1, 1, size=(len(tris), 3)).astype(np.float32)
    lights = [((0.5, 0.95, 0.5), (1.0, 1.0, 1.0), (1.0, 0.5, 0.25))]
    ref = vx.voxelize(tris, cols, n, lights, return_surface=True)
    got = run_voxelize(checked, str(tmp_path), tris, cols, n, lights, surface=surface)
    assert np.array_equal(got[0][..., 3], ref[0][..., 3].astype(np.float32)) and got[0][..., 3].sum() >= pixels / 3
    for g, r in zip(got, ref):
        assert np.abs(g[..., :3] - r[..., :3]).max() <= 1e-5 * np.abs(r[..., :3]).max()
