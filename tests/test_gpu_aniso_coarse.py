"""Anisotropic levels of at most 8 texels a side are built in one launch: grids whose
levels above 0 all are (n = 8: level 1 by itself, then the coarse ones), one with a
level of its own before them, and one whose top level is the only coarse one."""
import numpy as np
import pytest

import paper_2104_00618_amd as vct
from oracle import vct_aniso as va
from scenes import random_grid
from tests.test_gpu_aniso import decoded, gpu_aniso

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,levels", [(8, None), (32, None), (32, 3), (32, 2)])
def test_coarse_levels_match_oracle(n, levels):
    base = random_grid(n, seed=500 + n, alpha_max=0.8)
    pyr, g = gpu_aniso(base, n, levels)
    ref = va.build_aniso_mips(base, g.levels)
    got = decoded(pyr, g)
    # every level adds the rounding of 3 sums and an FMA on values below 2
    for d in range(6):
        for lv in range(1, g.levels):
            np.testing.assert_allclose(got[d][lv], ref[d][lv], rtol=0, atol=lv * 4e-7)
