"""Small and large frames take different kernels.  Through the checked CPU builds, small
frames run both: those that spread a tile's cones over waves, and those of large
frames, with every texel and accumulator index checked, and with the same bits."""
import numpy as np
import pytest

from scenes import ConeParams, cone_set, make_workload, random_gbuffer, random_grid, random_material, scene_lights
from tests.hostemu.driver import run_case
from tests.test_host_emulation import _params, checked, sanitized  # noqa: F401  (the build fixtures)


def _both(monkeypatch, binary, d, *args, **kw):
    monkeypatch.delenv("VCT_EMU_SPLIT_TILES", raising=False)
    split = run_case(binary, str(d / "split"), *args, **kw)
    monkeypatch.setenv("VCT_EMU_SPLIT_TILES", "0")
    whole = run_case(binary, str(d / "whole"), *args, **kw)
    names = [k for k in ("trace", "save", "grad", "grad_recompute", "grad_noalloc", "shade") if k in split]
    for k in names:
        assert np.isfinite(split[k]).all() and np.abs(split[k]).max() > 0, k
        assert np.array_equal(split[k].view(np.uint32), whole[k].view(np.uint32)), k
    assert np.array_equal(split["grad_recompute"].view(np.uint32), split["grad"].view(np.uint32))
    return names


@pytest.mark.parametrize("n,levels,shape,cones,dtype,aniso", [
    (16, None, (1, 17, 16), "six", "f32", False),    # a tile of one row below a full one
    (16, 2, (1, 13, 7), "five", "bf16", False),
    (8, None, (1, 9, 17), "five", "f32", True),
    (8, None, (1, 8, 8), "five", "f16", True),
    (1, None, (1, 9, 11), "six", "f32", False),
])
def test_both_kernels_give_the_same_bits(checked, tmp_path, monkeypatch, n, levels, shape, cones, dtype, aniso):  # noqa: F811
    pr, nr, cam = random_gbuffer(*shape, seed=6, n=max(n, 8))
    gout = np.random.default_rng(7).normal(size=shape + (8,)).astype(np.float32)
    names = _both(monkeypatch, checked, tmp_path, random_grid(n, seed=5, alpha_max=0.4), pr, nr, cam, _params(cones),
                  levels=levels, dtype=dtype, aniso=aniso, gout=gout, recompute=True, noalloc=True,
                  shade=scene_lights(3), material=random_material(shape, seed=8))
    assert len(names) == 6


def test_both_kernels_run_clean_under_the_sanitizers(sanitized, tmp_path, monkeypatch):  # noqa: F811
    w = make_workload("c3fd", h=8, w=9, views=1)
    gout = np.random.default_rng(7).normal(size=(1, 8, 9, 8)).astype(np.float32)
    _both(monkeypatch, sanitized, tmp_path, w.base, w.pos_rough, w.normal, w.cam_pos, w.params, gout=gout,
          recompute=True, shade=scene_lights(2), material=random_material((1, 8, 9), seed=1))


@pytest.mark.parametrize("cones,spec,occ", [("none", True, False), ("none", False, True), ("one", False, False),
                                            ("one", False, True), ("five", True, False), ("none", False, False)])
def test_the_scatter_pass_marches_the_cones_that_are_on(checked, tmp_path, monkeypatch, cones, spec, occ):  # noqa: F811
    """Any of a pixel's cones may be off, down to none: the others' workgroups are all there
    (in parts: the frame is small) and the gradient has the bits of the other kernel."""
    d, w = (np.zeros((0, 3), np.float32), np.zeros(0, np.float32)) if cones == "none" else cone_set("five")
    p = ConeParams(d[:1] if cones == "one" else d, w[:1] if cones == "one" else w, alpha_thresh=0.99, enable_spec=spec,
                   enable_occ=occ)
    pr, nr, cam = random_gbuffer(1, 9, 10, seed=6, n=8)
    gout = np.random.default_rng(7).normal(size=(1, 9, 10, 8)).astype(np.float32)
    args = (random_grid(8, seed=5, alpha_max=0.4), pr, nr, cam, p)
    monkeypatch.delenv("VCT_EMU_SPLIT_TILES", raising=False)
    split = run_case(checked, str(tmp_path / "split"), *args, gout=gout, recompute=True)
    monkeypatch.setenv("VCT_EMU_SPLIT_TILES", "0")
    whole = run_case(checked, str(tmp_path / "whole"), *args, gout=gout, recompute=True)
    for k in ("trace", "save", "grad", "grad_recompute"):
        assert np.array_equal(split[k].view(np.uint32), whole[k].view(np.uint32)), k
    assert (np.abs(split["grad"]).max() > 0) == (cones != "none" or spec or occ)
