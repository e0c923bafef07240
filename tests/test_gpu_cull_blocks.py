"""The culling tests on the matrix cores (blocks of 32 daughters, half
precision with every error on the passing side) against the navigators that
evaluate every daughter, bit for bit: daughter counts around the blocks'
edges, lines through the corners of boxes (where a dropped pair would show: a
box touches its bounding sphere there), geometries of very small and very
large units, daughters out of the tests' range, points far away or not
numbers, and volumes that are not culled because most lines meet most
daughters. The widening of r^2 that makes the tests conservative is checked
on the CPU with the tests' arithmetic restated in numpy."""
import numpy as np
import pytest

from paper_1312_0816_amd import workloads as W

BLOCK_EDGES = [1, 2, 8, 15, 16, 17, 31, 32, 33, 48, 49, 64, 65, 96, 129]


# ------------------------------------------------------------------ on the CPU

def _half_toward_zero(a):
    """float32 to half precision toward zero, as float32."""
    h = a.astype(np.float16)
    over = np.abs(h.astype(np.float32)) > np.abs(a)
    h = np.where(over, np.nextafter(h, np.float16(0)), h)
    return h.astype(np.float32)


def _split(a):
    a = np.asarray(a, np.float32)
    hi = _half_toward_zero(a)
    return hi, _half_toward_zero(a - hi)


def _filter(p, e, T, r, back, bound, sign):
    """The test's left side (passes when negative) for tracks (3, n) and as
    many daughters (3, n), (n,) in its units, every sum of products moved by
    4 x 2^-22 of its terms' magnitudes against passing (sign +1)."""
    f32 = np.float32
    e = e.astype(f32)
    start = (p.astype(f32) - f32(back) * e).astype(f32)
    tt = (T * T).sum(0)
    n = tt - r * r - 2.0 ** -15 * ((256.0 + back) ** 2 + tt)
    Th, Tl = _split(-2.0 * T.astype(f32))
    nh, nl = _split(n.astype(f32) / f32(64))
    ph, pl = _split(start)
    eh, el = _split(f32(0.5) * e)
    c = (start * start).sum(0, dtype=f32) / f32(64)
    pe = (start * e).sum(0, dtype=f32) / f32(64)

    def product(vh, vl, const, rest):
        ch, cl = _split(const)
        terms = [Th * vh, Th * vl, Tl * vh, [64.0 * ch, 64.0 * cl] + rest]
        flat = np.concatenate([np.stack(list(t)).astype(np.float64) for t in terms])
        return flat.sum(0) + sign * bound * np.abs(flat).sum(0)

    g = product(ph, pl, c, [64.0 * nh, 64.0 * nl])
    b = product(eh, el, pe, [])
    return g + b * np.abs(b) + sign * 2.0 ** -23 * (np.abs(g) + b * b)


@pytest.mark.parametrize("seed,size", [(1, 256.0), (2, 256.0), (3, 40.0), (4, 512.0)])
def test_no_line_that_meets_a_sphere_is_dropped(seed, size):
    """Half-lines tangent to culling spheres, or just inside them, from starts
    within the mother's radius (256 units): all pass, whatever way the sums
    are rounded; lines well outside (by 2 % of the mother) mostly do not."""
    rng = np.random.default_rng(seed)
    n = 200000
    p = rng.normal(size=(3, n))
    p *= 256.0 * rng.uniform(0, 1, n) ** (1 / 3) / np.linalg.norm(p, axis=0)
    T = rng.normal(size=(3, n))
    T *= size * rng.uniform(0, 1, n) ** (1 / 6) / np.linalg.norm(T, axis=0)
    r = 2.0 ** rng.uniform(-8, 5, n)
    back = float(r.max()) + 0.25
    w = T - p
    dist = np.linalg.norm(w, axis=0)
    side = np.cross(w.T, rng.normal(size=(n, 3))).T
    side /= np.linalg.norm(side, axis=0)
    for scale, wanted in ((1.0, True), (0.9, True), (None, False)):
        # a direction whose line is `off` from the centre, towards it
        off = np.minimum(r * scale if scale else r + 6.0, dist)
        s = off / dist
        e = np.sqrt(1 - s * s) * (w / dist) + s * side
        e /= np.linalg.norm(e, axis=0)
        f = _filter(p, e, T, r, back, 4 * 2.0 ** -22, 1.0)
        if wanted:
            assert (f < 0).all(), (scale, int((f >= 0).sum()), float(f.max()))
        else:
            far = dist > r + 6.0
            assert (f[far] >= 0).mean() > 0.9


# ------------------------------------------------------------------ on the GPU

@pytest.fixture(scope="module")
def gv():
    import torch
    from paper_1312_0816_amd import geonav
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    geonav.load_library()
    return geonav


def _bits(a):
    """Bits of an output, one pattern for every NaN."""
    a = a.cpu().numpy()
    return np.where(np.isnan(a), np.nan, a).view(np.int64) if a.dtype == np.float64 else a


def _boxes(rng, nd, unit=1.0, half=200.0, cells=6, kinds=(W.BOX,)):
    """A box mother (200 units) with nd rotated daughters in distinct cells of
    a 6^3 grid."""
    width = 2 * half / cells
    at = rng.choice(cells ** 3, nd, replace=False)
    c = (np.stack([at % cells, at // cells % cells, at // cells ** 2], axis=1) + 0.5) * width - half
    pars = np.zeros((nd, W.NPAR))
    kind = np.array([kinds[i % len(kinds)] for i in range(nd)], np.int32)
    bound = np.zeros(nd)
    for i in range(nd):
        par, rb = W._draw_daughter(rng, int(kind[i]))
        f = 0.9 * (width / 2) / max(rb, width / 2)
        keep = par.size if kind[i] in (W.BOX, W.TUBE, W.CONE) else None
        par = par * (f if keep else 1.0)
        pars[i, :par.size] = par * unit if keep else par
        bound[i] = rb * f * unit
    rots = np.stack([W.euler_zxz(*a) for a in rng.uniform(0, 6.28, (nd, 3))])
    return W.Volume(W.BOX, np.array([half * unit] * 3 + [0.0, 0.0]), kind, pars, rots, c * unit, bound)


def _corner_tracks(rng, vol, n, half, offsets=None):
    """Lines aimed at corners of the box daughters, on them and to both sides
    of them by 1e-9 and 1e-4 of the mother."""
    k = rng.integers(0, vol.nd, n)
    corner = rng.choice([-1.0, 1.0], (n, 3)) * vol.pars[k][:, :3]
    q = np.einsum("nij,nj->ni", vol.rots[k].reshape(-1, 3, 3), corner) + vol.trs[k]
    if offsets is not None:
        q = q + offsets[k]
    q = q + half * rng.choice([0.0, 1e-9, -1e-9, 1e-4, -1e-4], (n, 1)) * rng.normal(size=(n, 3))
    o = rng.uniform(-half, half, (n, 3))
    d = q - o
    d /= np.linalg.norm(d, axis=1)[:, None]
    return np.ascontiguousarray(np.concatenate([o.T, d.T]))


def _same(gv, vol, tr, offsets=None):
    """Every entry point on one volume with culling on and off: equal bits."""
    import torch
    g = gv.Geometry([vol])
    t = torch.from_numpy(tr).cuda()
    o, d = t[:3].contiguous(), t[3:].contiguous()
    offs = None if offsets is None else torch.from_numpy(offsets).cuda()
    gh = torch.from_numpy(np.random.default_rng(3).normal(size=(3, tr.shape[1]))).cuda()
    out = {}
    for cull in (True, False):
        g.culling = cull
        res = list(gv.geo_navigate_basket(g, 0, o, d, offs, hitpt=True))
        res += [gv.geo_navigate_safety(g, 0, o, offs), gv.geo_locate(g, 0, o, offs)]
        res += [x for x in gv.geo_navigate_backward(g, 0, o, d, offs, None, gh) if x is not None]
        if vol.nd <= 64:
            extra = [torch.empty_like(o), torch.empty_like(o), torch.empty((vol.nd, 3), dtype=o.dtype, device=o.device)]
            gv.geo_navigate_backward_noalloc(g, 0, o, d, offs, None, gh, *extra)
            res += extra
        if offs is None:
            n = tr.shape[1]
            for cfg in ((1, 0), (2, 0), (4, 0), (8, 0), (4, 4)):
                g.set_launch_config(*cfg)
                res += list(gv.geo_navigate_batched(g, [0, 0, 0], [0, n // 3, n // 2],
                                                    [n // 3, n // 2 - n // 3, n - n // 2], t))
        torch.cuda.synchronize()
        out[cull] = [_bits(x) for x in res]
    g.close()
    for i, (a, b) in enumerate(zip(out[True], out[False])):
        assert np.array_equal(a, b), (i, int((a != b).sum()))
    return out[True]


@pytest.mark.gpu
@pytest.mark.parametrize("nd", BLOCK_EDGES)
@pytest.mark.parametrize("with_offsets", [False, True])
def test_lines_through_box_corners(gv, nd, with_offsets):
    rng = np.random.default_rng(100 + nd)
    vol = _boxes(rng, nd)
    offs = rng.uniform(-0.5, 0.5, (nd, 3)) if with_offsets else None
    tr = _corner_tracks(rng, vol, 3001, 200.0, offs)
    res = _same(gv, vol, tr, offs)
    assert (res[1] >= 0).any()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 511, 513])
def test_ragged_tiles(gv, n):
    rng = np.random.default_rng(n)
    vol = _boxes(rng, 33, kinds=(W.BOX, W.TUBE, W.CONE, W.TUBS, W.CONS, W.PCON))
    _same(gv, vol, W.tracks_uniform_in_mother(rng, vol, n))


@pytest.mark.gpu
def test_baskets_of_many_rounds(gv):
    """2^20 + 77 tracks: four rounds per wavefront, the last tile ragged."""
    rng = np.random.default_rng(9)
    vol = _boxes(rng, 40)
    _same(gv, vol, W.tracks_uniform_in_mother(rng, vol, (1 << 20) + 77))


@pytest.mark.gpu
@pytest.mark.parametrize("unit", [1e-90, 1e-12, 1e-4, 1e5, 1e30, 1e60])
def test_units(gv, unit):
    """The same geometry in very small and very large units (the culling
    radius's absolute part of 1e-6 then outweighs the mother, or vanishes)."""
    rng = np.random.default_rng(7)
    vol = _boxes(rng, 20, unit=unit)
    tr = _corner_tracks(rng, vol, 1001, 200.0 * unit)
    tr[3:] *= max(unit, 1e-20)
    _same(gv, vol, tr)


@pytest.mark.gpu
def test_daughters_out_of_the_tests_range(gv):
    """A daughter larger than the mother, one far outside it, and offsets that
    move daughters out of range or are not numbers."""
    rng = np.random.default_rng(17)
    vol = _boxes(rng, 12)
    vol.pars[3, :3] = 3000.0
    vol.trs[3] = [0.0, 0.0, 4000.0]
    vol.trs[5] = [5000.0, 0.0, 0.0]
    tr = W.tracks_uniform_in_mother(rng, vol, 2000)
    tr = np.concatenate([tr, _corner_tracks(rng, vol, 2000, 200.0)], axis=1)
    tr = np.ascontiguousarray(tr)
    _same(gv, vol, tr)
    offs = rng.uniform(-1, 1, (12, 3))
    offs[2] = [900.0, 0.0, 0.0]
    offs[3] = [0.0, 0.0, -3000.0]
    offs[7] = 1e200
    _same(gv, vol, tr, offs)


@pytest.mark.gpu
@pytest.mark.parametrize("mother", [W.BOX, W.TUBE])
def test_starts_outside_and_not_numbers(gv, mother):
    """Points far outside the mother, infinite or not a number; zero, huge and
    undefined directions: the same bits with culling on and off."""
    rng = np.random.default_rng(23)
    vol = _boxes(rng, 18, kinds=(W.BOX, W.TUBE, W.CONE, W.TUBS, W.CONS, W.PCON))
    if mother == W.TUBE:
        vol.mother_kind, vol.mother_par = W.TUBE, np.array([0.0, 400.0, 200.0, 0.0, 0.0])
    tr = W.tracks_uniform_in_mother(rng, _boxes(rng, 1), 1500)
    tr[:3, 100:200] *= 10.0
    tr[:3, 200:300] *= 1e7
    tr[0, 300:310] = np.inf
    tr[1, 310:320] = np.nan
    tr[3:, 330:340] = 0.0
    tr[3:, 340:350] *= 1e80
    tr[3:, 350:360] *= 1e-18
    tr[4, 360:370] = 0.0
    _same(gv, vol, tr)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1000, 4099])
def test_volumes_that_are_not_culled(gv, n):
    """The paper's toy detector (most lines meet most daughters) alone, and
    beside culled volumes in one batched call, launched and replayed, with
    segments and polycones in the geometry and without."""
    import torch
    rng = np.random.default_rng(n)
    paper = W.paper_toy_detector()
    tr = W.paper_toy_tracks(seed=n, n=n)
    _same(gv, paper, tr)
    for other in (W.toy_detector_volume(), W.mixed_detector_volume()):
        vols = [paper, other, W.grid_volume(np.random.default_rng(2), 3)]
        pool = np.concatenate([tr, W.tracks_in_mother(rng, other, n), W.tracks_in_mother(rng, vols[2], n)], axis=1)
        t = torch.from_numpy(np.ascontiguousarray(pool)).cuda()
        which = np.repeat([0, 1, 2, 0], [1, 1, 1, 1])
        offset, size = np.array([0, n, 2 * n, n // 2]), np.array([n // 2, n, n, n - n // 2])
        g = gv.Geometry(vols)
        g.culling = False
        want = [_bits(x) for x in gv.geo_navigate_batched(g, which, offset, size, t)]
        g.culling = True
        for cfg in ((1, 0), (4, 0), (8, 0), (2, 4)):
            for graph in (False, True):
                g.set_launch_config(*cfg)
                g.batched_graph = graph
                got = gv.geo_navigate_batched(g, which, offset, size, t)
                torch.cuda.synchronize()
                for a, b in zip(want, got):
                    assert np.array_equal(a, _bits(b))
        s, h, counts = gv.geo_navigate_batched_census(g, which, offset, size, t)
        assert np.array_equal(_bits(s), want[0]) and np.array_equal(_bits(h), want[1])
        assert counts[gv.CENSUS_TRACKS] == 3 * n
        g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 23, 24, 25, 64])
def test_few_tracks_of_a_dense_volume(gv, n):
    """Up to 24 tracks such a volume is culled: every task, and batched
    baskets of both sides of the line, the same bits as the sequential loop."""
    import torch
    paper = W.paper_toy_detector()
    tr = torch.from_numpy(np.ascontiguousarray(W.paper_toy_tracks(seed=n, n=40 * n))).cuda()
    t = tr[:, :n].contiguous()
    o, d = t[:3].contiguous(), t[3:].contiguous()
    rng = np.random.default_rng(n)
    gs, gh = (torch.from_numpy(rng.uniform(-1, 1, k)).cuda() for k in ((n,), (3, n)))
    offs = torch.from_numpy(rng.uniform(-1, 1, (paper.nd, 3))).cuda()
    g = gv.Geometry([paper])
    perm = rng.permutation(40)
    out = {}
    for cull in (True, False):
        g.culling = cull
        res = []
        for f in (None, offs):
            res += [*gv.geo_navigate_basket(g, 0, o, d, f), gv.geo_navigate_safety(g, 0, t, f), gv.geo_locate(g, 0, t, f)]
        res += gv.geo_navigate_backward(g, 0, o, d, offs, gs, gh)
        res += gv.geo_navigate_batched(g, np.zeros(40, np.int32), perm * n, np.full(40, n), tr)
        out[cull] = [_bits(x) for x in res if x is not None]
    g.close()
    assert len(out[True]) == len(out[False])
    for a, b in zip(out[True], out[False]):
        assert np.array_equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("kinds", [(W.BOX,), (W.TUBE, W.CONE), (W.BOX, W.TUBE, W.CONE, W.TUBS, W.CONS, W.PCON)])
@pytest.mark.parametrize("nd", [7, 8, 32, 70])
def test_safety_near_daughters(gv, kinds, nd):
    """Points just outside, on and inside the daughters' bounding spheres,
    where the bound from the nearest daughter starts to count."""
    import torch
    rng = np.random.default_rng(1000 + nd)
    vol = _boxes(rng, nd, kinds=kinds)
    n = 5000
    k = rng.integers(0, nd, n)
    u = np.stack(W.isotropic(rng, n))
    r = vol.bound_r[k] * rng.choice([0.0, 0.3, 0.99, 1.0, 1.0 + 1e-6, 1.0 + 1e-5, 1.001, 1.1, 2.0, 4.0], n)
    p = torch.from_numpy(np.ascontiguousarray(vol.trs[k].T + r * u)).cuda()
    offs = torch.from_numpy(rng.uniform(-2, 2, (nd, 3))).cuda()
    g = gv.Geometry([vol])
    out = {}
    for cull in (True, False):
        g.culling = cull
        out[cull] = [_bits(gv.geo_navigate_safety(g, 0, p, f)) for f in (None, offs)]
    g.close()
    for a, b in zip(out[True], out[False]):
        assert np.array_equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("kinds", [(W.BOX, W.TUBE, W.CONE), (W.TUBE, W.CONS), (W.BOX, W.TUBE, W.CONE, W.TUBS, W.CONS, W.PCON)])
@pytest.mark.parametrize("nd", [5, 13, 44, 53, 54, 63, 64, 65])
def test_safety_records(gv, kinds, nd):
    """The daughters' records copied by a workgroup, around the counts where
    its copy takes one pass more and where it stops; workgroups and wavefronts
    that are full, nearly empty and empty; the same bits as the sequential loop."""
    import torch
    rng = np.random.default_rng(nd)
    vol = _boxes(rng, nd, kinds=kinds)
    tr = torch.from_numpy(W.tracks_uniform_in_mother(rng, vol, 1100)).cuda()
    offs = torch.from_numpy(rng.uniform(-2, 2, (nd, 3))).cuda()
    g = gv.Geometry([vol])
    for n in (1, 63, 64, 65, 192, 256, 257, 1100):
        p = tr[:3, :n].contiguous()
        out = {}
        for cull in (True, False):
            g.culling = cull
            out[cull] = [_bits(gv.geo_navigate_safety(g, 0, p, f)) for f in (None, offs)]
        for a, b in zip(out[True], out[False]):
            assert np.array_equal(a, b)
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("kinds", [(W.BOX, W.TUBE, W.CONE), (W.BOX, W.TUBE, W.CONE, W.TUBS, W.CONS, W.PCON)])
@pytest.mark.parametrize("n", [(7 << 16) - 1, 7 << 16, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, (1 << 20) + 255,
                               (1 << 20) + 1025, (1 << 21) + (1 << 20) + 300])
def test_adjoint_passes(gv, kinds, n):
    """The adjoint around the sizes from which a workgroup takes four passes
    at a time (and over its largest grid), against the same tracks in smaller
    baskets: tracks' gradients bit for bit, the offsets' to the rounding of
    differently grouped sums; culling on and off the same bits."""
    import torch
    rng = np.random.default_rng(n)
    vol = _boxes(rng, 33, kinds=kinds)
    m = 200003
    tr = torch.from_numpy(W.tracks_uniform_in_mother(rng, vol, m)).cuda().repeat(1, -(-n // m))[:, :n]
    o, d = tr[:3].contiguous(), tr[3:].contiguous()
    gs = torch.rand(n, dtype=o.dtype, device="cuda") - 0.5
    gh = torch.rand((3, n), dtype=o.dtype, device="cuda") - 0.5
    offs = torch.from_numpy(rng.uniform(-0.5, 0.5, (33, 3))).cuda()
    g = gv.Geometry([vol])
    out = {}
    for cull in (True, False):
        g.culling = cull
        out[cull] = [_bits(x) for x in gv.geo_navigate_backward(g, 0, o, d, offs, gs, gh)]
    for a, b in zip(out[True], out[False]):
        assert np.array_equal(a, b)
    g.culling = True
    parts = []
    for i in range(0, n, m):
        c = slice(i, min(i + m, n))
        parts.append(gv.geo_navigate_backward(g, 0, o[:, c].contiguous(), d[:, c].contiguous(), offs,
                                              gs[c].contiguous(), gh[:, c].contiguous()))
    for k in (0, 1):
        assert np.array_equal(out[True][k], _bits(torch.cat([p[k] for p in parts], dim=1)))
    off = sum(p[2] for p in parts).cpu().numpy()
    got = out[True][2].view(np.float64)
    # each entry is a sum of at most n terms: n eps of the terms' magnitudes
    # bounds the difference of two groupings; the terms are -c ds/dp, the
    # difference of g_o and ghit
    terms = (out[True][0].view(np.float64) - gh.cpu().numpy())
    assert np.abs(got - off).max() <= n * 2.3e-16 * np.abs(terms).sum(1).max()
    g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("kinds", [(W.BOX, W.TUBE, W.CONE), (W.BOX, W.TUBE, W.CONE, W.TUBS, W.CONS, W.PCON)])
@pytest.mark.parametrize("n", [(3 << 18) - 1, 3 << 18, (3 << 18) + 1, (3 << 18) + 257, (1 << 20) + 63])
def test_locate_rounds(gv, kinds, n):
    """Localization around the size from which a wavefront takes four rounds,
    points uniform in the mother and points crowded into the daughters (full
    queues in the middle of a round): culling on and off, and in smaller
    baskets, the same indices."""
    import torch
    rng = np.random.default_rng(n)
    vol = _boxes(rng, 40, kinds=kinds)
    m = 100003
    p = W.tracks_uniform_in_mother(rng, vol, m)[:3]
    k = rng.integers(0, vol.nd, m)
    crowd = vol.trs[k].T + 0.7 * vol.bound_r[k] * rng.uniform(-1, 1, (3, m))
    offs = torch.from_numpy(rng.uniform(-1, 1, (vol.nd, 3))).cuda()
    g = gv.Geometry([vol])
    for pts in (p, crowd, np.where(rng.uniform(size=m) < 0.5, p, 1.5 * crowd)):
        t = torch.from_numpy(np.ascontiguousarray(pts)).cuda().repeat(1, -(-n // m))[:, :n].contiguous()
        for f in (None, offs):
            out = {}
            for cull in (True, False):
                g.culling = cull
                out[cull] = gv.geo_locate(g, 0, t, f)
            assert torch.equal(out[True], out[False])
            g.culling = True
            parts = [gv.geo_locate(g, 0, t[:, i:i + m].contiguous(), f) for i in range(0, n, m)]
            assert torch.equal(out[True], torch.cat(parts))
    g.close()
