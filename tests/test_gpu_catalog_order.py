"""Stored order of uploaded catalogs (needs an MI355X for the upload): region,
then the Morton curve of the coordinates (21 bits each), then the point's
index, whatever number of host threads shared the sort.  The order is compared
with numpy's stable sort of the same keys."""

import numpy as np
import pytest

import oracle
import paper_1204_6630_amd as tp
import synthcat

pytestmark = pytest.mark.gpu


def _spread(v):
    r = np.zeros_like(v)
    for b in range(21):
        r |= (v >> np.uint64(b) & np.uint64(1)) << np.uint64(3 * b)
    return r


def _keys(xyz, lo, hi):
    q = [np.clip((c - lo) / (hi - lo) * 2097151.0, 0.0, 2097151.0).astype(np.uint64) for c in xyz]
    return _spread(q[0]) | _spread(q[1]) << np.uint64(1) | _spread(q[2]) << np.uint64(2)


@pytest.mark.parametrize("regions", [0, 1, 7, 1024])
@pytest.mark.parametrize("n", [1, 2, 4095, 8191, 8192, 12289, 70001])
def test_order_of_sky_and_box(n, regions):
    """Every third point is a copy of an earlier one (equal keys)."""
    g = synthcat.rng_for(99, n)
    ra, dec = synthcat.uniform_patch(n, (0.0, 90.0, -20.0, 60.0), g)
    ra[2::3], dec[2::3] = ra[: ra[2::3].size], dec[: dec[2::3].size]
    label = g.integers(0, max(1, regions), n).astype(np.int32)
    first = label if regions else np.zeros(n, np.int32)
    ctx = tp.Context(0)
    try:
        xyz = oracle.radec_to_xyz(ra, dec)
        a = ctx.upload_catalog_regions(ra, dec, label, regions) if regions else ctx.upload_catalog(ra, dec)
        assert np.array_equal(ctx.catalog_order(a), np.lexsort((np.arange(n), _keys(xyz, -1.0, 1.0), first)))
        box = tuple(3.0 * c for c in xyz)
        lo, hi = min(c.min() for c in box), max(c.max() for c in box)
        b = ctx.upload_catalog_3d_regions(*box, label, regions) if regions else ctx.upload_catalog_3d(*box)
        if hi > lo:
            assert np.array_equal(ctx.catalog_order(b), np.lexsort((np.arange(n), _keys(box, lo, hi), first)))
    finally:
        ctx.close()
