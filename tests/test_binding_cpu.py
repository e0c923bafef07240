"""The binding's argument marshalling without a GPU: the records that basket
lists and shapes become, field by field."""
import numpy as np
import pytest

from paper_1312_0816_amd import geonav as gv


@pytest.mark.parametrize("form", [list, np.asarray, lambda v: np.asarray(v, np.int32), lambda v: np.asarray(v)[::1]])
@pytest.mark.parametrize("nb", [0, 1, 7, 1000])
def test_basket_records(form, nb):
    rng = np.random.default_rng(nb)
    vol, off, n = (rng.integers(0, 1 << 20, nb).tolist() for _ in range(3))
    arr, count = gv._baskets(form(vol), form(off), form(n))
    assert count == nb and len(arr) == max(nb, 1) and arr._type_ is gv.GeoBasket
    assert [(b.volume, b._pad, b.offset, b.n) for b in arr[:nb]] == [(v, 0, o, k) for v, o, k in zip(vol, off, n)]


def test_basket_records_keep_what_is_out_of_range():
    """Negative and 64-bit values reach the library's own checks."""
    arr, _ = gv._baskets([-3, 2, 1], [-(1 << 40), 1 << 40, 5], [1 << 33, -1, 0])
    assert [(b.volume, b.offset, b.n) for b in arr] == [(-3, -(1 << 40), 1 << 33), (2, 1 << 40, -1), (1, 5, 0)]
    with pytest.raises(ValueError):
        gv._baskets([0, 1], [0], [1])


@pytest.mark.parametrize("m", [0, 1, 7, gv.NPAR, gv.NPAR + 1])
def test_shape_record(m):
    par = np.arange(1.0, m + 1.0)
    if m > gv.NPAR:
        with pytest.raises(ValueError):
            gv.make_shape(gv.GEO_PCON, par)
        return
    s = gv.make_shape(gv.GEO_CONS, par)
    assert s.kind == gv.GEO_CONS and list(s.par) == par.tolist() + [0.0] * (gv.NPAR - m)
