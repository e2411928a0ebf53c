"""Small and large frames take different kernels (cones spread over waves, or
one lane for all the cones of a pixel).  A frame's outputs are the same bits
either way: a small frame is compared with the corner of a frame that is past
both dispatch sizes (768 and 4096 tiles of 16x16 pixels) and empty elsewhere."""
import numpy as np
import pytest
import torch

import paper_2104_00618_amd as vct
from scenes import ConeParams, cone_set, random_gbuffer, random_grid, random_material, scene_lights

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


# tile edges of 8 and 16 pixels with remainders; one pixel; no diffuse cones,
# more cones than waves, cones switched off; lights from none to all
@pytest.mark.parametrize("h,w,cones,spec,occ,dtype,aniso,lights", [
    (1, 1, "five", True, True, "f32", False, 1),
    (8, 8, "six", True, False, "f16", False, 0),
    (9, 17, "five", False, True, "bf16", True, 3),
    (16, 23, "none", True, True, "f32", True, 2),
    (33, 15, "sixteen", True, True, "f32", False, 4),
    # (1, 4, 8 and 16 waves for one cone in the scatter pass: by the waves of the frame)
    (203, 210, "six", True, True, "f32", True, 1),
    (150, 163, "six", True, True, "bf16", False, 1),
    (105, 101, "six", True, True, "f16", True, 1),
])
def test_small_frame_same_bits_as_in_a_large_one(h, w, cones, spec, occ, dtype, aniso, lights):
    n = 16
    if cones == "none":
        d, wt = np.zeros((0, 3), np.float32), np.zeros(0, np.float32)
    elif cones == "sixteen":
        d = np.random.default_rng(3).normal(size=(16, 3)).astype(np.float32)
        d[:, 2] = np.abs(d[:, 2]) + 0.1
        wt = np.full(16, 1 / 16, np.float32)
    else:
        d, wt = cone_set(cones)
    p = ConeParams(d, wt, alpha_thresh=0.99, enable_spec=spec, enable_occ=occ)
    grid = vct.Grid(n, dtype=dtype, anisotropic=aniso)
    pyr = vct.build_mips(dev(random_grid(n, seed=5, alpha_max=0.6)), grid)
    pr, nr, cam = random_gbuffer(1, h, w, seed=6, n=n, invalid_frac=0.1)
    mat = random_material((1, h, w), seed=7)
    side = 16 * 64 + 1   # 65 x 65 tiles

    def embed(t):
        out = torch.zeros((1, side, side, t.shape[-1]), device=DEV)
        out[:, :h, :w] = t
        return out

    corner = lambda t: t[:, :h, :w]  # noqa: E731
    small = [dev(x) for x in (pr, nr, cam)]
    large = [embed(small[0]), embed(small[1]), small[2]]
    m_small = dev(mat)
    same = lambda a, b: torch.equal(a.contiguous().view(torch.int32), b.contiguous().view(torch.int32))  # noqa: E731
    assert same(vct.trace(pyr, grid, *small, p), corner(vct.trace(pyr, grid, *large, p)))
    out_s, st_s = vct.trace_save(pyr, grid, *small, p)
    out_l, st_l = vct.trace_save(pyr, grid, *large, p)
    assert same(out_s, corner(out_l))
    s = scene_lights(lights)
    assert same(vct.shade(pyr, grid, *small, m_small, p, s),
                corner(vct.shade(pyr, grid, *large, embed(m_small), p, s)))
    g = torch.randn(out_s.shape, generator=torch.Generator(device=DEV).manual_seed(8), device=DEV)
    g_large = embed(g)
    ref = vct.trace_backward_saved(pyr, grid, *small, p, st_s, g)
    assert same(ref, vct.trace_backward(pyr, grid, *small, p, g))
    assert same(ref, vct.trace_backward_saved(pyr, grid, *large, p, st_l, g_large))
    assert same(ref, vct.trace_backward(pyr, grid, *large, p, g_large))
    assert float(ref.abs().max()) > 0 or cones == "none"
