"""The order in which the adjoint sums the offset gradient: a row of partial sums
takes the passes of 256 tracks b, b + rows, b + 2 rows, ... (rows: at most 2048), each
pass's tracks daughter by daughter in track order, and the rows are added by a tree
over 256 threads. The sum is restated in numpy from the per-track gradients, bit for
bit, around the sizes at which a workgroup takes more passes together; culled, not
culled, of volumes in lockstep, and by the entry point that allocates nothing."""
import numpy as np
import pytest

from paper_1312_0816_amd import workloads as W

BLOCK, ROWS = 256, 2048


@pytest.fixture(scope="module")
def gv():
    import torch
    from paper_1312_0816_amd import geonav
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    geonav.load_library()
    return geonav


def _sum(hit, grad, nd):
    """Offset gradient of per-track contributions grad (3, n) to the daughter hit."""
    n = hit.size
    npass = -(-n // BLOCK)
    rows = min(npass, ROWS)
    # each pass's sum per daughter, track after track (a sum from 0 on)
    sums = np.zeros((npass, 3 * nd))
    where = np.flatnonzero(hit >= 0)
    for c in range(3):
        np.add.at(sums, (where // BLOCK, 3 * hit[where] + c), grad[c, where])
    part = np.zeros((rows, 3 * nd))
    for first in range(0, npass, rows):
        m = min(rows, npass - first)
        part[:m] += sums[first:first + m]
    acc = np.zeros((BLOCK, 3 * nd))
    for b in range(0, rows, BLOCK):
        m = min(BLOCK, rows - b)
        acc[:m] += part[b:b + m]
    w = BLOCK // 2
    while w > 0:
        acc[:w] += acc[w:2 * w]
        w //= 2
    return acc[0].reshape(nd, 3)


SIZES = [1000, (11 << 15) - 1, 11 << 15, (1 << 19) - 3, 1 << 19, (1 << 19) + 1, 5 << 17, (1 << 20) - 255, 1 << 20,
         (1 << 20) + 1, (1 << 20) + 513, (1 << 21) + 300]


@pytest.mark.gpu
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("detector", ["toy", "mixed", "paper"])
def test_order_of_the_sums(gv, detector, n):
    import torch
    rng = np.random.default_rng(n)
    vol = {"toy": W.toy_detector_volume, "mixed": W.mixed_detector_volume, "paper": W.paper_toy_detector}[detector]()
    m = 100003
    few = W.paper_toy_tracks(seed=n, n=m) if detector == "paper" else W.tracks_uniform_in_mother(rng, vol, m)
    tr = torch.from_numpy(few).cuda().repeat(1, -(-n // m))[:, :n]
    o, d = tr[:3].contiguous(), tr[3:].contiguous()
    gs = torch.from_numpy(rng.uniform(-1.0, 1.0, n)).cuda()
    offs = torch.from_numpy(rng.uniform(-0.5, 0.5, (vol.nd, 3))).cuda()
    g = gv.Geometry([vol])
    hit = gv.geo_navigate_basket(g, 0, o, d, offs)[1].cpu().numpy()
    out = []
    for cull in (True, False):
        g.culling = cull
        out.append([x.cpu().numpy() for x in gv.geo_navigate_backward(g, 0, o, d, offs, gs, None)])
    g.culling = True
    extra = [torch.empty_like(o), torch.empty_like(o), torch.empty((vol.nd, 3), dtype=o.dtype, device=o.device)]
    gv.geo_navigate_backward_noalloc(g, 0, o, d, offs, gs, None, *extra)
    out.append([x.cpu().numpy() for x in extra])
    no_sum = [torch.empty_like(o), torch.empty_like(o)]
    gv.geo_navigate_backward_noalloc(g, 0, o, d, offs, gs, None, *no_sum, None)
    g.close()
    # without an upstream gradient of the hit point a track's share of its
    # daughter's gradient is the negative of its own
    want = _sum(hit, -out[0][0], vol.nd)
    for res in out:
        assert np.array_equal(res[0], out[0][0]) and np.array_equal(res[1], out[0][1])
        assert np.array_equal(res[2], want)
    for k in (0, 1):
        assert np.array_equal(no_sum[k].cpu().numpy(), out[0][k])
