"""Cone sets as the binding takes them: lists, arrays and tensors, with one number an element
also where that is an array of its own (a column of weights)."""
import types

import numpy as np
import pytest
import torch

from paper_2104_00618_amd.binding import cone_params
from scenes import ConeParams, cone_set


@pytest.mark.filterwarnings("ignore::DeprecationWarning")
@pytest.mark.parametrize("form", [
    lambda d, w: (d, w), lambda d, w: (d.tolist(), w.tolist()), lambda d, w: (torch.from_numpy(d), torch.from_numpy(w)),
    lambda d, w: (d, w[:, None]), lambda d, w: (torch.from_numpy(d), torch.from_numpy(w)[:, None]),
    lambda d, w: (d[:, :, None], w), lambda d, w: (list(d), list(w)),
    lambda d, w: (np.concatenate([d, d], 1), w)])
def test_forms_of_a_cone_set_give_the_same_cones(form):
    d, w = (np.asarray(x, np.float32) for x in cone_set("five"))
    p = ConeParams(d, w)
    q = types.SimpleNamespace(**{k: getattr(p, k) for k in dir(p) if not k.startswith("_") and not callable(getattr(p, k))})
    q.diffuse_dirs, q.diffuse_weights = form(d, w)
    assert bytes(cone_params(q)) == bytes(cone_params(p))
