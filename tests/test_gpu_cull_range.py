"""Culling at the ends of its range: daughters whose radii lie around the
largest that the half-precision tests take, and geometries of very many
volumes."""
import numpy as np
import pytest

from paper_1312_0816_amd import workloads as W


@pytest.fixture(scope="module")
def gv():
    import torch
    from paper_1312_0816_amd import geonav
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    geonav.load_library()
    return geonav


def _placed(mother, daughters):
    """A volume of unrotated daughters (kind, parameters, place)."""
    pars = np.zeros((len(daughters), W.NPAR))
    for i, (_, p, _) in enumerate(daughters):
        pars[i, :len(p)] = p
    return W.Volume(W.BOX, np.array(list(mother) + [0.0, 0.0]), np.array([k for k, _, _ in daughters], np.int32), pars,
                    np.tile(np.eye(3).reshape(9), (len(daughters), 1)), np.array([t for _, _, t in daughters], float),
                    np.zeros(len(daughters)))


@pytest.mark.gpu
@pytest.mark.parametrize("radius", [511.9, 512.05, 512.1, 512.3])
def test_safety_radii_around_the_largest(gv, radius):
    """The tests' unit is 1/256 of the mother's radius, 1 here, and they take
    radii of up to 512 units. A polycone with its planes far from its origin,
    of `radius` units: its sphere is the nearest of all, its solid is not, and
    a small box beyond the sphere's reach sets the Safety. A tube of just under
    512 units is present. The same bits with culling on and off."""
    import torch
    mother = (1.0, 1.0, float(np.sqrt(256.0 ** 2 - 2.0)))
    a = 511.9 / np.sqrt(2.0)
    z = float(np.sqrt(radius ** 2 - 400.0))
    d = [(W.TUBE, [0.0, a, a], (-500.0, 0.0, 0.0)),
         (W.PCON, W.pcon_par(0.0, 2 * np.pi, [(-z, 0.0, 20.0), (-z + 1.0, 0.0, 20.0)]), (0.0, 0.0, 0.0)),
         (W.BOX, [2.9, 2.9, 2.9], (80.0, 0.0, 0.0))]
    d += [(W.BOX, [0.5, 0.5, 0.5], (-200.0 - 10.0 * k, 0.0, 0.0)) for k in range(9)]
    vol = _placed(mother, d)
    # the polycone's planes face away from the points: at -x
    vol.rots[1] = np.array([0.0, 0.0, 1.0, 0.0, 1.0, 0.0, -1.0, 0.0, 0.0])
    rng = np.random.default_rng(1)
    p = rng.uniform(-20.0, 20.0, (3, 2000))
    p[0] += 700.0
    t = torch.from_numpy(p).cuda()
    offs = torch.zeros((len(d), 3), dtype=torch.float64, device="cuda")
    g = gv.Geometry([vol])
    out = {}
    for cull in (True, False):
        g.culling = cull
        out[cull] = [gv.geo_navigate_safety(g, 0, t, f).cpu().numpy() for f in (None, offs)]
    g.close()
    nearest = np.linalg.norm(np.maximum(np.abs(p - np.array([[80.0], [0.0], [0.0]])) - 2.9, 0.0), axis=0)
    for a_, b_ in zip(out[True], out[False]):
        assert np.abs(b_ - nearest).max() < 1e-9
        assert np.array_equal(a_, b_)


@pytest.mark.gpu
def test_many_volumes(gv):
    """70,001 volumes of none, one or 33 daughters (more than one dimension of
    a grid takes): each volume's culling blocks are its own."""
    import torch
    nvol = 70001
    rng = np.random.default_rng(4)
    none = W.Volume(W.BOX, np.array([10.0, 10.0, 10.0, 0.0, 0.0]))
    one = [_placed((10.0, 10.0, 10.0), [(W.BOX, [0.2, 0.2, 0.2], tuple(rng.uniform(-8, 8, 3)))]) for _ in range(7)]
    many = _placed((10.0, 10.0, 10.0), [(W.BOX, [0.2, 0.2, 0.2], tuple(rng.uniform(-8, 8, 3))) for _ in range(33)])
    vols = [none if i % 5 == 3 else (many if i % 1000 == 999 else one[i % 7]) for i in range(nvol)]
    vols[-3:] = [many, none, one[0]]
    g = gv.Geometry(vols)
    t = torch.from_numpy(W.tracks_uniform_in_mother(rng, one[0], 40)).cuda()
    o, d = t[:3].contiguous(), t[3:].contiguous()
    for v in (0, 1, 3, 999, 65535, 65536, 69999, nvol - 3, nvol - 2, nvol - 1):
        out = {}
        for cull in (True, False):
            g.culling = cull
            res = [*gv.geo_navigate_basket(g, v, o, d), gv.geo_navigate_safety(g, v, o), gv.geo_locate(g, v, o)]
            res += list(gv.geo_navigate_batched(g, [v], [0], [40], t))
            out[cull] = [x.cpu().numpy() for x in res if x is not None]
        for a, b in zip(out[True], out[False]):
            assert np.array_equal(a, b)
    g.close()
