"""Paths of the voxelizer's raster pass: slots named by the fragment's pixel (bounding
boxes of at most n^3 pixels in all) or taken from a counter (more), and lanes that find
their triangle among the 64 offsets a wave holds or past them (many triangles without
pixels in between)."""
import numpy as np
import pytest

from oracle import vct_voxelize as vx
from tests.test_gpu_voxelize import LIGHTS, gpu_voxelize, mesh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,copies,empty", [(1, 1, 0), (2, 1, 0), (4, 30, 0), (16, 1, 63), (16, 3, 64), (32, 1, 500)])
def test_voxelize_paths_match_oracle(n, copies, empty):
    tris, cols = mesh(5, extra=20)
    tris, cols = np.tile(tris, (copies, 1, 1)), np.tile(cols, (copies, 1))
    if empty:   # degenerate triangles after every third one
        keep = np.arange(len(tris)) // 3 * (3 + empty) + np.arange(len(tris)) % 3
        t2 = np.full((int(keep.max()) + 1 + empty, 3, 3), 0.25, np.float32)
        c2 = np.ones((len(t2), 3), np.float32)
        t2[keep], c2[keep] = tris, cols
        tris, cols = t2, c2
    base, nrm, alb = gpu_voxelize(tris, cols, n, surface=True)
    ref, cnt, rn, ra = vx.voxelize(tris, cols, n, LIGHTS, return_counts=True, return_surface=True)
    np.testing.assert_array_equal(base[..., 3], (cnt > 0).astype(np.float32))
    assert np.abs(base[..., :3] - ref[..., :3]).max() <= 1e-5 * max(np.abs(ref[..., :3]).max(), 1e-30)
    assert np.abs(nrm[..., :3] - rn[..., :3]).max() <= 1e-6 and np.abs(alb[..., :3] - ra[..., :3]).max() <= 1e-6
