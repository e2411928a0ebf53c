"""The directional mip adjoint takes the levels of at most 8 texels a side in one launch:
pyramids of which all levels are that small (the base among them), some, the top one
only, or none, in each storage type (16-bit ones against the stored values)."""
import numpy as np
import pytest

import paper_2104_00618_amd as vct
from oracle import vct_aniso as va
from scenes import ConeParams, cone_set, random_gbuffer, random_grid
from tests.test_gpu_aniso import _check_grad, decoded, dev, gpu_aniso

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("n,levels", [(8, None), (8, 1), (32, None), (16, 2), (64, 3)])
def test_directional_adjoint_matches_oracle(n, levels, dtype):
    base = random_grid(n, seed=700 + n, alpha_max=0.35)
    pr, nr, cam = random_gbuffer(1, 19, 21, seed=n, n=n)
    d, w = cone_set("five")
    p = ConeParams(d, w, alpha_thresh=0.99)
    pyr, g = gpu_aniso(base, n, levels, dtype)
    am = decoded(pyr, g)
    gout = np.random.default_rng(n).normal(size=(1, 19, 21, 8)).astype(np.float32)
    _, info = va.trace_aniso(am, pr, nr, cam, p, return_info=True)
    gout[info["ambiguous"]] = 0.0
    t = [dev(x) for x in (pr, nr, cam)]
    _, state = vct.trace_save(pyr, g, *t, p)
    got = vct.trace_backward_saved(pyr, g, *t, p, state, dev(gout)).cpu().numpy()
    _check_grad(got, va.trace_backward_aniso(am, pr, nr, cam, p, gout), f"{n}^3 levels {levels} {dtype}")
