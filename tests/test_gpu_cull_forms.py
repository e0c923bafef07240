"""Volumes whose lines meet many daughters: the culling tests in FP64, and the calls
and tiles of few tracks on volumes that are walked in lockstep. Every form gives the
bits of the navigators that evaluate every daughter; the census counts what passes
the tests."""
import numpy as np
import pytest

from paper_1312_0816_amd import workloads as W
from tests.test_gpu_cull_blocks import _bits, _same

BASIC = (W.BOX, W.TUBE, W.CONE)
EVERY = (W.BOX, W.TUBE, W.CONE, W.TUBS, W.CONS, W.PCON)


@pytest.fixture(scope="module")
def gv():
    import torch
    from paper_1312_0816_amd import geonav
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    geonav.load_library()
    return geonav


def _spheres(nd, ratio, kinds, seed=1):
    """Daughters at random places (they may overlap) whose bounding spheres meet
    `ratio` of the lines through a box mother of half-length 200."""
    rng = np.random.default_rng(seed)
    c = rng.uniform(-100.0, 100.0, (nd, 3))
    kind, pars, rots, _, bound = W._place_daughters(rng, c, 60.0, kinds)
    size = np.sqrt(ratio * 24.0 * 200.0 ** 2 / (4.0 * np.pi))
    for i in range(nd):
        f, k = size / bound[i], int(kind[i])
        lo, hi = {W.TUBS: (0, 3), W.CONS: (0, 5)}.get(k, (3, 3 + 3 * int(pars[i, 2])) if k == W.PCON else (0, 5))
        pars[i, lo:hi] *= f
    return W.Volume(W.BOX, np.array([200.0] * 3 + [0.0, 0.0]), kind, pars, rots, c, np.full(nd, size))


def _pairs(gv, vol, tr):
    """Pairs that pass the culling tests, by the census, and those whose half-line
    meets the daughter's bounding sphere."""
    import torch
    n = tr.shape[1]
    g = gv.Geometry([vol])
    counts = gv.geo_navigate_batched_census(g, [0], [0], [n], torch.from_numpy(tr).cuda())[2]
    g.close()
    exact = 0
    for k in range(vol.nd):
        r = vol.bound_r[k]
        if vol.kinds[k] == W.PCON:  # (the library's sphere holds the polycone's bounding cylinder)
            z, _, rmax = W.pcon_planes(vol.pars[k])
            r = np.hypot(np.abs(z).max(), rmax.max())
        w = tr[:3] - vol.trs[k][:, None]
        b = np.minimum((w * tr[3:]).sum(0), 0.0)
        exact += int(((w * w).sum(0) - b * b <= r * r).sum())
    return int(sum(int(c) for c in counts[:14])), exact


@pytest.mark.gpu
@pytest.mark.parametrize("kinds", [BASIC, EVERY])
@pytest.mark.parametrize("nd", [8, 33])
@pytest.mark.parametrize("ratio", [0.06, 0.12])
def test_pairs_of_large_spheres(gv, kinds, nd, ratio):
    """Spheres behind a start are left out where they are large and many (lines with
    spheres that meet up to 8 % of them, of every kind; 16 % of box, tube and cone)."""
    vol = _spheres(nd, min(ratio, 0.07) if kinds is EVERY else ratio, kinds)
    tr = W.tracks_uniform_in_mother(np.random.default_rng(nd), vol, 6000)
    passed, exact = _pairs(gv, vol, tr)
    assert exact <= passed <= 1.01 * exact


@pytest.mark.gpu
@pytest.mark.parametrize("kinds", [BASIC, EVERY])
@pytest.mark.parametrize("nd", [3, 8, 33, 70])
@pytest.mark.parametrize("ratio", [0.02, 0.035, 0.06, 0.12, 0.3, 0.8])
def test_many_pairs(gv, kinds, nd, ratio):
    """From few pairs per track to nearly all: queues and lists that fill within a
    round, every entry point, with offsets and without."""
    rng = np.random.default_rng(nd)
    vol = _spheres(nd, ratio, kinds)
    _same(gv, vol, W.tracks_uniform_in_mother(rng, vol, 1500))
    _same(gv, vol, W.tracks_uniform_in_mother(rng, vol, 777), rng.uniform(-20.0, 20.0, (nd, 3)))


@pytest.mark.gpu
@pytest.mark.parametrize("kinds", [BASIC, EVERY])
def test_many_pairs_of_large_baskets(gv, kinds):
    """The same from the sizes on at which a wavefront takes several rounds."""
    vol = _spheres(40, 0.06, kinds)
    _same(gv, vol, W.tracks_uniform_in_mother(np.random.default_rng(9), vol, (1 << 20) + 77))


@pytest.mark.gpu
@pytest.mark.parametrize("n", [15, 16, 17, 39, 40, 41, 47, 48, 49])
def test_few_tracks_of_volumes_in_lockstep(gv, n):
    """Around the numbers of tracks up to which such volumes are culled all the
    same, alone and as baskets beside other volumes, of every launch shape."""
    import torch
    paper, rng = W.paper_toy_detector(), np.random.default_rng(n)
    tr = np.ascontiguousarray(W.paper_toy_tracks(seed=n, n=n))
    _same(gv, paper, tr)
    _same(gv, paper, tr, rng.uniform(-1.0, 1.0, (paper.nd, 3)))
    for other in (W.toy_detector_volume(), W.mixed_detector_volume(), _spheres(20, 0.06, BASIC)):
        pool = np.concatenate([W.paper_toy_tracks(seed=n, n=12 * n), W.tracks_uniform_in_mother(rng, other, 4 * n)],
                              axis=1)
        t = torch.from_numpy(np.ascontiguousarray(pool)).cuda()
        order = rng.permutation(16)
        which = np.where(order < 12, 0, 1)
        g = gv.Geometry([paper, other])
        out = {}
        for cull in (False, True):
            g.culling = cull
            out[cull] = []
            for cfg in ((1, 0), (2, 0), (4, 0), (8, 0), (1, 4), (2, 4), (4, 4)):
                g.set_launch_config(*cfg)
                out[cull] += [_bits(x) for x in gv.geo_navigate_batched(g, which, order * n, np.full(16, n), t)]
        g.close()
        for a, b in zip(out[True], out[False]):
            assert np.array_equal(a, b)
