"""The units of the culling tests, for daughters that are small against their mother:
the pairs that pass, and the bits of the navigators that evaluate every daughter."""
import numpy as np
import pytest

from paper_1312_0816_amd import workloads as W
from tests.test_gpu_cull_blocks import _corner_tracks, _same
from tests.test_gpu_cull_forms import BASIC, EVERY, _pairs


@pytest.fixture(scope="module")
def gv():
    import torch
    from paper_1312_0816_amd import geonav
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    geonav.load_library()
    return geonav


def _in_mother(vol, half, shift=(0.0, 0.0, 0.0)):
    """The daughters of vol, moved, in a box mother of another size."""
    return W.Volume(W.BOX, np.array([half] * 3 + [0.0, 0.0]), vol.kinds, vol.pars, vol.rots,
                    vol.trs + np.asarray(shift, float), vol.bound_r)


def _join(a, b):
    return W.Volume(a.mother_kind, a.mother_par, np.concatenate([a.kinds, b.kinds]), np.concatenate([a.pars, b.pars]),
                    np.concatenate([a.rots, b.rots]), np.concatenate([a.trs, b.trs]),
                    np.concatenate([a.bound_r, b.bound_r]))


@pytest.mark.gpu
@pytest.mark.parametrize("kinds", [BASIC, EVERY])
@pytest.mark.parametrize("factor", [10.0, 30.0, 100.0, 1000.0, 1e5])
@pytest.mark.parametrize("shift", [0.0, 0.6])
def test_pairs_in_a_large_mother(gv, kinds, factor, shift):
    """A detector in a mother `factor` times its size, at its centre or off it, the
    tracks in the detector and far outside it: at most 1.3 times the pairs whose
    line meets a bounding sphere are evaluated."""
    base = W.toy_detector_volume() if kinds is BASIC else W.mixed_detector_volume()
    at = np.array([shift, -shift, 0.5 * shift]) * 200.0 * factor
    vol = _in_mother(base, 200.0 * factor, at)
    rng = np.random.default_rng(int(factor))
    tr = W.tracks_in_mother(rng, base, 6000)
    tr[:3] += at[:, None]
    # and tracks from all over the mother, aimed at daughters
    far = rng.uniform(-200.0 * factor, 200.0 * factor, (3, 2000))
    d = vol.trs[rng.integers(0, vol.nd, 2000)].T + rng.normal(size=(3, 2000)) * 30.0 - far
    far = np.concatenate([far, d / np.linalg.norm(d, axis=0)])
    passed, exact = _pairs(gv, vol, np.ascontiguousarray(np.concatenate([tr, far], axis=1)))
    assert exact <= passed <= 1.3 * exact


@pytest.mark.gpu
@pytest.mark.parametrize("factor", [10.0, 100.0, 3000.0, 1e6, 1e9])
@pytest.mark.parametrize("nd", [5, 33])
def test_large_mothers(gv, factor, nd):
    """Lines through the corners of box daughters (which touch their bounding
    spheres) from starts near them and all over a mother of `factor` times the
    detector's size, with offsets that leave the daughters where they are, move some
    out of the detector and move some out of the mother: every entry point."""
    rng = np.random.default_rng(nd + int(factor))
    cells = rng.choice(216, nd, replace=False)
    c = (np.stack([cells % 6, cells // 6 % 6, cells // 36], axis=1) - 2.5) * 66.0
    pars = np.zeros((nd, W.NPAR))
    pars[:, :3] = rng.uniform(4.0, 18.0, (nd, 3))
    rots = np.stack([W.euler_zxz(*a) for a in rng.uniform(0.0, 6.28, (nd, 3))])
    small = W.Volume(W.BOX, np.array([200.0] * 3 + [0.0, 0.0]), np.full(nd, W.BOX, np.int32), pars, rots, c,
                     np.linalg.norm(pars[:, :3], axis=1))
    at = np.array([0.3, -0.5, 0.1]) * 200.0 * factor
    vol = _in_mother(small, 200.0 * factor, at)
    near = _corner_tracks(rng, small, 1500, 200.0)
    near[:3] += at[:, None]
    far = _corner_tracks(rng, vol, 1500, 200.0 * factor)
    tr = np.ascontiguousarray(np.concatenate([near, far], axis=1))
    tr[3:, ::7] *= 1e-3
    tr[3:, 1::11] *= -1.0
    res = _same(gv, vol, tr)
    assert (res[1] >= 0).any()
    offs = rng.uniform(-0.5, 0.5, (nd, 3))
    _same(gv, vol, tr, offs)
    offs[::3] += rng.uniform(-400.0, 400.0, offs[::3].shape)
    offs[1::4] *= 3.0 * factor
    _same(gv, vol, tr, offs)


@pytest.mark.gpu
def test_clusters_far_apart(gv):
    """Two detectors at the ends of a mother 200 times their size, which one unit
    does not resolve: pairs and bits."""
    base = W.mixed_detector_volume()
    half = 200.0 * 200.0
    vol = _join(_in_mother(base, half, (0.9 * half, 0.0, 0.0)), _in_mother(base, half, (-0.9 * half, 0.0, 0.0)))
    tr = W.tracks_in_mother(np.random.default_rng(3), base, 4000)
    tr[0] += np.where(np.arange(4000) % 2 == 0, 0.9 * half, -0.9 * half)
    passed, exact = _pairs(gv, vol, tr)
    assert exact <= passed <= 1.1 * exact
    _same(gv, vol, tr)
    _same(gv, vol, tr, np.random.default_rng(4).uniform(-1.0, 1.0, (vol.nd, 3)))
