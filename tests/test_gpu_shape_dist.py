"""The polycone's distances over large baskets (tracks that need evaluating
are queued, the others known at once) against the same tracks in baskets
below the sizes from which that form is taken, bit for bit: sizes around the
thresholds and with ragged last tiles, every polycone variant, uncut and cut,
points all inside, all outside and mixed, lines tangent to the bounding
sphere, and undefined inputs."""
import numpy as np
import pytest

from paper_1312_0816_amd import workloads as W

pytestmark = pytest.mark.gpu
SMALL = 500_003


@pytest.fixture(scope="module")
def gv():
    import torch
    from paper_1312_0816_amd import geonav
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    geonav.load_library()
    return geonav


def _same(gv, par, t):
    import torch
    n = t.shape[1]
    for q in (gv.GEO_DIST_IN, gv.GEO_DIST_OUT):
        big = gv.geo_shape_query(W.PCON, par, q, t)
        parts = [gv.geo_shape_query(W.PCON, par, q, t[:, i:i + SMALL].contiguous()) for i in range(0, n, SMALL)]
        a, b = big.cpu().numpy(), torch.cat(parts).cpu().numpy()
        assert np.array_equal(np.where(np.isnan(a), np.nan, a).view(np.int64),
                              np.where(np.isnan(b), np.nan, b).view(np.int64)), (q, n)


def _tile(tr, n):
    """n tracks repeating tr (6, m), the repeats scaled a little in place."""
    import torch
    t = torch.from_numpy(tr).cuda()
    reps = -(-n // t.shape[1])
    t = t.repeat(1, reps)[:, :n].clone()
    t[:3] *= 1.0 + 1e-3 * torch.linspace(-1, 1, n, dtype=t.dtype, device=t.device)
    return t


@pytest.mark.parametrize("variant", range(len(W.PCON_VARIANTS) + 1))
def test_variants(gv, variant):
    par = (W.PCON_VARIANTS + [W.SUITE_SHAPES[W.PCON]])[variant]
    _, _, tr = W.shape_suite_c1(W.PCON, n=100003, seed=variant, par=par)
    _same(gv, par, _tile(tr, (1 << 21) + 77))


@pytest.mark.parametrize("n", [(1 << 20) - 1, 1 << 20, (1 << 20) + 1, (1 << 21) - 1, 1 << 21, (1 << 21) + 1,
                               (1 << 21) + 255, (1 << 21) + 1023])
def test_sizes(gv, n):
    par = W.PCON_VARIANTS[3]
    _, _, tr = W.shape_suite_c1(W.PCON, n=50021, seed=5, par=par)
    _same(gv, par, _tile(tr, n))


@pytest.mark.parametrize("which", ["inside", "outside", "tangent", "undefined"])
def test_inputs(gv, which):
    par = W.PCON_VARIANTS[2]
    _, _, tr = W.shape_suite_c1(W.PCON, n=200003, seed=6, par=par)
    rng = np.random.default_rng(6)
    if which in ("inside", "outside"):
        import torch
        held = gv.geo_shape_query(W.PCON, par, gv.GEO_CONTAINS, torch.from_numpy(tr).cuda()).cpu().numpy() == 1
        tr = np.ascontiguousarray(tr[:, held if which == "inside" else ~held])
    elif which == "tangent":
        z, _, rout = W.pcon_planes(par)
        far = np.hypot(rout.max(), np.abs(z).max())
        n = tr.shape[1]
        u = np.stack(W.isotropic(rng, n))
        side = np.cross(u.T, rng.normal(size=(n, 3))).T
        side /= np.linalg.norm(side, axis=0)
        off = far * rng.choice([1.0, 1.0 + 1e-7, 1.0 + 1e-6, 1.0 + 2e-6, 0.9], n)
        d = -u * 10.0 ** rng.uniform(-18, 60, n)
        tr = np.ascontiguousarray(np.concatenate([u * 10.0 ** rng.uniform(0, 9, n) + side * off, d]))
    else:
        tr[:, 100:120] = np.nan
        tr[0, 200:220] = np.inf
        tr[3:, 300:330] = 0.0
        tr[4, 400:420] = 0.0
        tr[5, 500:520] = np.nan
        tr[3:, 600:620] *= 1e95
        tr[3:, 700:720] *= 1e-25
    t = _tile(tr, (1 << 21) + 333)
    _same(gv, par, t)
