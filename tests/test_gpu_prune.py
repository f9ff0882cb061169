"""GPU parity of pruned launches at the edges of the block test (needs an
MI355X).

One call of the test covers 64 aligned blocks of 64 columns: column counts
one below, at and one above a block and 64 of them, chunks that start inside
a block (auto-pairs, row ranges), rows that do and do not fill a wavefront.
Counts are integers: they equal the oracle's, no tolerance.
"""

import numpy as np
import pytest

import oracle
import paper_1204_6630_amd as tp
import synthcat

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tp.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("prec", [tp.FP32_CHORD, tp.FP64])
@pytest.mark.parametrize("max_cols", [256, 65536])
@pytest.mark.parametrize("n", [63, 64, 65, 257, 4095, 4096, 4097, 8257])
def test_blocks_of_the_sky(ctx, n, max_cols, prec):
    """513 rows of a 3 x 3 deg patch against n columns of a 60 x 60 deg one,
    bins of 7 and 33 degrees (64 neighbouring columns span 8 to 15; the
    columns reach past both ends)."""
    g = synthcat.rng_for(97, n)
    d = synthcat.uniform_patch(513, (30.0, 33.0, -3.0, 0.0), g)
    r = synthcat.uniform_patch(n, (10.0, 70.0, -30.0, 30.0), g)
    e = np.array([5.0, 12.0, 45.0])
    xd, xr = oracle.radec_to_xyz(*d), oracle.radec_to_xyz(*r)
    a, b = ctx.upload_catalog(*d), ctx.upload_catalog(*r)
    try:
        ctx.set_tuning(prune=1, max_cols=max_cols, rows_per_lane=4)
        ctx.stats(reset=True)
        assert np.array_equal(ctx.count(tp.DR, a, e, cat_b=b, precision=prec),
                              oracle.count(oracle.DR, xd, e, b_xyz=xr))
        if n >= 4095:
            st = ctx.stats(reset=True)
            assert 0 < st.pruned_pairs < st.pairs
        if n <= 4097:
            assert np.array_equal(ctx.count(tp.DD, b, e, precision=prec), oracle.count(oracle.DD, xr, e))
        if n in (257, 4097):
            o = ctx.catalog_order(b)
            sb = tuple(np.ascontiguousarray(c[o]) for c in xr)
            lo, hi = n // 3, n // 3 + (n + 1) // 2
            assert np.array_equal(ctx.count(tp.DD, b, e, row_begin=lo, row_end=hi, precision=prec),
                                  oracle.count(oracle.DD, sb, e, row_begin=lo, row_end=hi))
    finally:
        ctx.set_tuning()
        ctx.release_catalog(a)
        ctx.release_catalog(b)


@pytest.mark.parametrize("prec", [tp.FP32_CHORD, tp.FP64])
@pytest.mark.parametrize("scale", [1e-155, 1.0, 1e9])
@pytest.mark.parametrize("n", [65, 4097])
def test_blocks_of_a_box(ctx, n, scale, prec):
    """The same in 3-D, edges from 0 on, at scales whose squares are subnormal
    numbers, ordinary and large."""
    g = synthcat.rng_for(97, 9000 + n)
    p, q = synthcat.box_uniform(513, 100.0, g), synthcat.box_uniform(n, 100.0, g)
    e = np.array([0.0, 20.0, 60.0, 110.0]) * scale
    x, y = tuple(c * scale for c in p.xyz()), tuple(c * scale for c in q.xyz())
    a, b = ctx.upload_catalog_3d(*x), ctx.upload_catalog_3d(*y)
    try:
        ctx.set_tuning(prune=1)
        assert np.array_equal(ctx.count(tp.DR, a, e, cat_b=b, precision=prec), oracle.count3d(oracle.DR, x, e, b_xyz=y))
        assert np.array_equal(ctx.count(tp.DD, b, e, precision=prec), oracle.count3d(oracle.DD, y, e))
    finally:
        ctx.set_tuning()
        ctx.release_catalog(a)
        ctx.release_catalog(b)
