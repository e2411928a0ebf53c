"""The scatter pass marches each cone again; its samples have to be those of the forward
whose end state it divides by, or a cone that saturates (alpha_thresh = 1) passes A = 1
too early and its gradient is not finite."""
import numpy as np
import pytest
import torch

from scenes import ConeParams, cone_set
from scenes.cornell import make_scene, render_gbuffer
from tests.test_fixed_point import run_program


def test_remarch_sets_up_the_forwards_cones(tmp_path):
    run_program(tmp_path, "remarch_case.cpp")


# A saturating cone's last samples are known to their order only (a transmittance that
# float32 holds in steps of 2^-24 divides them); on opaque solids they are a few in a
# hundred of the gradient.
@pytest.mark.gpu
@pytest.mark.parametrize("n,aniso", [(16, False), (32, False), (32, True)])
def test_gradient_of_saturating_cones(n, aniso):
    import oracle
    import paper_2104_00618_amd as vct
    from oracle import vct_aniso as va
    sc = make_scene(n, seed=3, n_boxes=(2, 2), n_spheres=(1, 1), avoid=[(0.5, 0.5, 0.8)])
    base = np.asarray(sc.base, np.float32)
    pr, nr = (np.asarray(t, np.float32)[None] for t in render_gbuffer(sc, (0.5, 0.5, 0.8), (0.5, 0.45, 0.2), 48, 64))
    cam = np.array([[0.5, 0.5, 0.8]], np.float32)
    d, w = cone_set("five")
    p = ConeParams(d, w, alpha_thresh=1.0)
    gout = np.random.default_rng(4).normal(size=(1, 48, 64, 8)).astype(np.float32)
    if aniso:
        mips = va.build_aniso_mips(base)
        ref = va.trace_backward_aniso(mips, pr, nr, cam, p, gout)
    else:
        ref = oracle.trace_backward(oracle.build_mips(base), pr, nr, cam, p, gout)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")  # noqa: E731
    grid = vct.Grid(n, anisotropic=aniso)
    pyr = vct.build_mips(t(base), grid)
    view = [t(x) for x in (pr, nr, cam)]
    _, st = vct.trace_save(pyr, grid, *view, p)
    got = vct.trace_backward_saved(pyr, grid, *view, p, st, t(gout))
    assert torch.equal(got, vct.trace_backward(pyr, grid, *view, p, t(gout)))
    err = np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"{n}^3 {'directional' if aniso else 'isotropic'}: relative error {err:.2e}", flush=True)
    assert err <= 5e-2
