"""Backward passes over grids with values that are not finite, through the checked
CPU build: every index that the scatter pass forms stays inside the accumulator,
whatever the sums are.  (One texel or one channel that overflows float16, a NaN
channel; one level and all; isotropic and directional pyramids.)"""
import numpy as np
import pytest

from scenes import random_gbuffer, random_grid
from tests.hostemu.driver import run_case
from tests.test_host_emulation import _params, checked  # noqa: F401  (the build fixture)


def _grid(n, what):
    base = random_grid(n, seed=5, alpha_max=0.6)
    if what == "one texel":
        base[n // 2, n // 2, n // 2, 0] = 1e5
    elif what == "red":
        base[..., 0] = 1e5
    else:
        base[..., 0] = np.nan
    return base


@pytest.mark.parametrize("levels", [1, None])
@pytest.mark.parametrize("aniso", [False, True])
@pytest.mark.parametrize("dtype,what", [("f16", "one texel"), ("f16", "red"), ("f32", "nan")])
def test_scatter_stays_in_the_accumulator(checked, tmp_path, dtype, what, aniso, levels):  # noqa: F811
    _backward(checked, tmp_path, dtype, what, aniso, levels)


@pytest.mark.parametrize("aniso", [False, True])
@pytest.mark.parametrize("dtype,what", [("f16", "one texel"), ("f16", "red"), ("f32", "nan")])
def test_a_colour_that_is_not_finite_shows_in_the_gradient(checked, tmp_path, dtype, what, aniso):  # noqa: F811
    """One such channel of one cone is enough, as where all three are: the gradient is NaN everywhere."""
    res = _backward(checked, tmp_path, dtype, what, aniso, None)
    assert not np.isfinite(res["save"]).all()
    assert np.isnan(res["grad"]).all()


def _backward(checked, tmp_path, dtype, what, aniso, levels):  # noqa: F811
    n = 8
    pr, nr, cam = random_gbuffer(1, 8, 8, seed=6, n=n)
    gout = np.random.default_rng(7).normal(size=(1, 8, 8, 8)).astype(np.float32)
    return run_case(checked, str(tmp_path), _grid(n, what), pr, nr, cam, _params(), dtype=dtype, aniso=aniso,
                    levels=levels, gout=gout)
