"""Calls on volumes of few daughters around the sizes at which a basket walks them in
lockstep and a localization takes more rounds: the bits of the navigators that
evaluate every daughter."""
import numpy as np
import pytest

from paper_1312_0816_amd import workloads as W
from tests.test_gpu_cull_blocks import _same


@pytest.fixture(scope="module")
def gv():
    import torch
    from paper_1312_0816_amd import geonav
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    geonav.load_library()
    return geonav


@pytest.mark.gpu
@pytest.mark.parametrize("nd,n", [(1, (1 << 19) - 1), (2, (1 << 19) - 1), (2, 1 << 19), (3, (1 << 19) - 1),
                                  (11, 3 << 18), (12, (3 << 18) - 1), (12, 3 << 18)])
def test_few_daughters(gv, nd, n):
    rng = np.random.default_rng(nd)
    vol = W.grid_volume(rng, nd)
    res = _same(gv, vol, W.tracks_uniform_in_mother(rng, vol, n))
    assert (res[1] >= 0).any()
