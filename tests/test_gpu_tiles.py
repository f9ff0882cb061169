"""GPU parity of the FP32 tiles at the edges of their shapes (needs an MI355X).

A wavefront takes 64, 128 or 256 rows in groups of 32 against 64 columns at a
time, in two tiles of 32; a lane holds one column against 16 consecutive rows.
Row and column counts one below, at and one above each of these, and row
ranges that start anywhere, must count every pair once, in the slot of the
exact rule.  Counts are integers: they equal the oracle's, no tolerance.
"""

import numpy as np
import pytest

import oracle
import paper_1204_6630_amd as tp
import synthcat

pytestmark = pytest.mark.gpu

SIZES = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 513, 1025]


@pytest.fixture(scope="module")
def ctx():
    c = tp.Context(0)
    yield c
    c.close()


def _stored(ctx, cat, xyz):
    o = ctx.catalog_order(cat)
    return tuple(np.ascontiguousarray(c[o]) for c in xyz)


@pytest.mark.parametrize("rows", [0, 2, 4])
@pytest.mark.parametrize("n", SIZES)
def test_ragged_sky_catalogs(ctx, n, rows):
    """n rows against n + 31 columns on a 10 x 10 deg patch, 12 log bins to
    the patch's size: near and far tiles, masked diagonals and tails."""
    g = synthcat.rng_for(96, n)
    fp = (20.0, 30.0, -5.0, 5.0)
    d, r = synthcat.uniform_patch(n, fp, g), synthcat.uniform_patch(n + 31, fp, g)
    e = synthcat.log_edges(0.01, 8.0, 12)
    xd, xr = oracle.radec_to_xyz(*d), oracle.radec_to_xyz(*r)
    a, b = ctx.upload_catalog(*d), ctx.upload_catalog(*r)
    try:
        ctx.set_tuning(rows_per_lane=rows)
        assert np.array_equal(ctx.count(tp.DD, a, e), oracle.count(oracle.DD, xd, e))
        assert np.array_equal(ctx.count(tp.DR, a, e, cat_b=b), oracle.count(oracle.DR, xd, e, b_xyz=xr))
        if n > 2:
            sa = _stored(ctx, a, xd)
            lo, hi = n // 3, n - n // 5
            assert np.array_equal(ctx.count(tp.DD, a, e, row_begin=lo, row_end=hi),
                                  oracle.count(oracle.DD, sa, e, row_begin=lo, row_end=hi))
    finally:
        ctx.set_tuning()
        ctx.release_catalog(a)
        ctx.release_catalog(b)


@pytest.mark.parametrize("n", [33, 257, 1025])
@pytest.mark.parametrize("scale", [1e-30, 1.0, 3e9])
def test_ragged_boxes_of_any_scale(ctx, n, scale):
    """3-D points and edges times a scale factor: the tiles bring coordinates
    into f16's range by a power of two of their own.  The box lies off the
    origin, so the rows' mean carries the distances."""
    g = synthcat.rng_for(96, 5000 + n)
    p = synthcat.box_uniform(n, 100.0, g, origin=37.0)
    q = synthcat.box_uniform(2 * n + 1, 100.0, g, origin=37.0)
    e = np.concatenate([[0.0], np.geomspace(0.5, 120.0, 17)]) * scale
    x, y = tuple(c * scale for c in p.xyz()), tuple(c * scale for c in q.xyz())
    a, b = ctx.upload_catalog_3d(*x), ctx.upload_catalog_3d(*y)
    try:
        assert np.array_equal(ctx.count(tp.DD, a, e), oracle.count3d(oracle.DD, x, e))
        assert np.array_equal(ctx.count(tp.DR, a, e, cat_b=b), oracle.count3d(oracle.DR, x, e, b_xyz=y))
    finally:
        ctx.release_catalog(a)
        ctx.release_catalog(b)


@pytest.mark.parametrize("nbins", [1, 7, 46, 125, 126, 200, 256])
def test_bins_finer_than_a_tile(ctx, nbins):
    """Bins from wider than a tile to far narrower (one slot, one edge, a few
    edges and lookups), linear so that far bins are the narrow ones, on rows
    in upload order (attached: no Morton order, tiles spread over the sky)
    and in Morton order."""
    import torch
    g = synthcat.rng_for(96, 9000 + nbins)
    d, r = synthcat.uniform_patch(1500, synthcat.OCTANT, g), synthcat.uniform_patch(1700, synthcat.OCTANT, g)
    e = np.linspace(1e-3, 75.0, nbins + 1)
    xd, xr = oracle.radec_to_xyz(*d), oracle.radec_to_xyz(*r)
    ref = oracle.count(oracle.DR, xd, e, b_xyz=xr)
    a, b = ctx.upload_catalog(*d), ctx.upload_catalog(*r)
    t = torch.from_numpy(np.stack(xd)).cuda()
    c = ctx.attach_catalog(t)
    try:
        assert np.array_equal(ctx.count(tp.DR, a, e, cat_b=b), ref)
        assert np.array_equal(ctx.count(tp.DR, c, e, cat_b=b), ref)
    finally:
        for k in (a, b, c):
            ctx.release_catalog(k)


def test_pairs_at_every_edge_and_at_zero(ctx):
    """Columns at theta = e_k (1 +- 10^-s), s = 2..12, from rows in a tight
    clump, coincident and antipodal points among them: the matrix-core
    distances are off by up to a few 1e-7 of the distance, so most of these
    pairs lie within their error of an edge and are settled by differences
    or the FP64 rule."""
    g = synthcat.rng_for(96, 1)
    e = synthcat.log_edges(0.05, 150.0, 14)
    c = np.array([0.6, 0.64, np.sqrt(1 - 0.36 - 0.4096)])
    t1 = np.cross(c, [0.0, 0.0, 1.0])
    t1 /= np.linalg.norm(t1)
    t2 = np.cross(c, t1)
    rows = c[None, :] + g.normal(0.0, 1e-9, size=(300, 3))
    rows /= np.linalg.norm(rows, axis=1)[:, None]
    cols = [c, -c]
    for k in e:
        for s in range(2, 13):
            for sign in (1.0, -1.0):
                th, ph = np.radians(k * (1.0 + sign * 10.0 ** -s)), g.uniform(0, 2 * np.pi)
                cols.append(np.cos(th) * c + np.sin(th) * (np.cos(ph) * t1 + np.sin(ph) * t2))
    cols = np.array(cols)
    cols /= np.linalg.norm(cols, axis=1)[:, None]
    a, b = rows.T.copy(), cols.T.copy()
    ca, cb = ctx.upload_catalog_xyz(*a), ctx.upload_catalog_xyz(*b)
    try:
        ctx.stats(reset=True)
        assert np.array_equal(ctx.count(tp.DR, ca, e, cat_b=cb), oracle.count(oracle.DR, a, e, b_xyz=b))
        assert ctx.stats(reset=True).exact > 0
        assert np.array_equal(ctx.count(tp.DR, cb, e, cat_b=ca), oracle.count(oracle.DR, b, e, b_xyz=a))
    finally:
        ctx.release_catalog(ca)
        ctx.release_catalog(cb)


@pytest.mark.parametrize("prec", [tp.FP32_CHORD, tp.FP64])
@pytest.mark.parametrize("n", [500, 5632, 5633, 12000])
def test_items_of_several_queues(ctx, n, prec):
    """One block per compute unit and 256-column units: fewer work items than
    wavefronts, a few more, and several times as many, dealt to counters that
    run dry at different times."""
    g = synthcat.rng_for(98, n)
    fp = (20.0, 40.0, -10.0, 10.0)
    d, r = synthcat.uniform_patch(n, fp, g), synthcat.uniform_patch(5000, fp, g)
    e = synthcat.log_edges(0.05, 15.0, 9)
    xd, xr = oracle.radec_to_xyz(*d), oracle.radec_to_xyz(*r)
    a, b = ctx.upload_catalog(*d), ctx.upload_catalog(*r)
    try:
        ctx.set_tuning(rows_per_lane=2, max_cols=256, blocks_per_cu=1)
        ctx.stats(reset=True)
        assert np.array_equal(ctx.count(tp.DR, a, e, cat_b=b, precision=prec), oracle.count(oracle.DR, xd, e, b_xyz=xr))
        assert ctx.stats(reset=True).pairs == n * 5000
    finally:
        ctx.set_tuning()
        ctx.release_catalog(a)
        ctx.release_catalog(b)


def test_launches_leave_nothing_behind(ctx):
    """Requests of different slot counts, empty ones and repeated ones after
    each other on one stream: each finds its histogram copies and queues
    cleared by the one before."""
    g = synthcat.rng_for(98, 77)
    fp = (20.0, 30.0, -5.0, 5.0)
    d = synthcat.uniform_patch(1500, fp, g)
    xd = oracle.radec_to_xyz(*d)
    a = ctx.upload_catalog(*d)
    try:
        for nbins in (256, 3, 40, 1, 126, 256):
            e = np.linspace(0.1, 9.0, nbins + 1)
            want = oracle.count(oracle.DD, xd, e)
            assert not ctx.count(tp.DD, a, e, row_begin=7, row_end=7).any()
            for prec in (tp.FP32_CHORD, tp.FP64, tp.FP32_CHORD):
                assert np.array_equal(ctx.count(tp.DD, a, e, precision=prec), want)
    finally:
        ctx.release_catalog(a)


@pytest.mark.parametrize("last", [89.0, 90.0, 91.0, 180.0])
def test_fp64_steps_beyond_an_edge_near_90_degrees(ctx, last):
    """FP64 steps beyond a last edge below 90 degrees are told by the dot
    product itself, others by 1 - d: points all over the sphere, both signs of
    the dot product, edges on either side of where the test changes."""
    g = synthcat.rng_for(98, int(last))
    d = synthcat.uniform_patch(700, (0.0, 360.0, -90.0, 90.0), g)
    r = synthcat.uniform_patch(1300, (0.0, 360.0, -90.0, 90.0), g)
    e = np.array([10.0, 45.0, last])
    xd, xr = oracle.radec_to_xyz(*d), oracle.radec_to_xyz(*r)
    a, b = ctx.upload_catalog(*d), ctx.upload_catalog(*r)
    try:
        assert np.array_equal(ctx.count(tp.DR, a, e, cat_b=b, precision=tp.FP64), oracle.count(oracle.DR, xd, e, b_xyz=xr))
        assert np.array_equal(ctx.count(tp.DD, b, e, precision=tp.FP64), oracle.count(oracle.DD, xr, e))
    finally:
        ctx.release_catalog(a)
        ctx.release_catalog(b)


CORNERS = [(x, y, z) for x in (-1.0, 1.0) for y in (-1.0, 1.0) for z in (-1.0, 1.0)]


@pytest.mark.parametrize("rows", [0, 2, 4])
@pytest.mark.parametrize("edges", [(1e-9, 2.0), (0.0, 1e-9, 2.0), (1e-9, 0.5, 1.5), (1e-9, 0.5, 2.0),
                                   (0.0, 1e-9, 2e-9, 0.5, 1.1)])
@pytest.mark.parametrize("around", [[(1.0, 0.0, 0.0), (-1.0, 0.0, 0.0)], CORNERS], ids=["pair", "cube"])
def test_column_at_the_rows_mean(ctx, around, edges, rows):
    """Rows placed symmetrically about a column, and a first edge below the
    FP32 band (its band reaches 0): the column's slot has no lower edge and no
    width.  Rows in upload order and shuffled, in multiples of every
    wavefront's rows; DD with the mean itself among the points."""
    e = np.array(edges)
    g = synthcat.rng_for(96, 31)
    for n in (64, 128, 256, 512):
        p = np.tile(np.array(around), (n // len(around), 1))
        for q in (p, g.permutation(p), np.concatenate([p, np.zeros((64, 3))]), np.concatenate([p[:-1], np.zeros((1, 3))])):
            x, y = tuple(q.T.copy()), tuple(np.zeros((3, 1)))
            a, b = ctx.upload_catalog_3d(*x), ctx.upload_catalog_3d(*y)
            try:
                ctx.set_tuning(rows_per_lane=rows)
                assert np.array_equal(ctx.count(tp.DR, a, e, cat_b=b), oracle.count3d(oracle.DR, x, e, b_xyz=y))
                assert np.array_equal(ctx.count(tp.DD, a, e), oracle.count3d(oracle.DD, x, e))
                assert np.array_equal(ctx.count(tp.DR, b, e, cat_b=a), oracle.count3d(oracle.DR, y, e, b_xyz=x))
            finally:
                ctx.set_tuning()
                ctx.release_catalog(a)
                ctx.release_catalog(b)


@pytest.mark.parametrize("prec", [tp.FP32_CHORD, tp.FP64])
@pytest.mark.parametrize("edges", [(10.0, 20.0), (0.0, 20.0, 1e140), (2.5, 1e30), (1e-9, 1e9)])
@pytest.mark.parametrize("extent", [0.0, 1.0])
def test_3d_edges_beyond_every_pair(ctx, extent, edges, prec):
    """Edges of which the first positive one lies further than any two points
    of the catalogs, catalogs of one place and empty ones: every entry point
    that compiles 3-D edges."""
    g = synthcat.rng_for(96, 47)
    x, y = tuple(extent * g.uniform(-0.5, 0.5, (3, 300))), tuple(extent * g.uniform(-0.5, 0.5, (3, 77)))
    e = np.array(edges)
    a, b = ctx.upload_catalog_3d(*x), ctx.upload_catalog_3d(*y)
    none = ctx.upload_catalog_3d(*np.zeros((3, 0)))
    try:
        dd, dr = oracle.count3d(oracle.DD, x, e), oracle.count3d(oracle.DR, x, e, b_xyz=y)
        assert np.array_equal(ctx.count(tp.DD, a, e, precision=prec), dd)
        assert np.array_equal(ctx.count(tp.DR, a, e, cat_b=b, precision=prec), dr)
        assert not ctx.count(tp.DD, none, e, precision=prec).any()
        got = ctx.count_batch([(tp.DD, a, -1), (tp.DR, a, b)], e, precision=prec)
        assert np.array_equal(got[0], dd) and np.array_equal(got[1], dr)
        assert np.array_equal(ctx.wait(ctx.submit(tp.DR, a, e, cat_b=b, precision=prec), e.size + 1), dr)
    finally:
        for c in (a, b, none):
            ctx.release_catalog(c)


@pytest.mark.parametrize("spread", [1e-6, 1e-4, 1e-2, 0.3])
def test_pairs_within_the_error_of_an_edge(ctx, spread):
    """The matrix cores' squared distance is trusted beyond e = 2^-24 (24 b^2
    + 640 r^2) of an edge (b: the column's distance from the rows' mean, r the
    rows' radius; a constant term is below 3e-13).  Every column lies within 3
    e of an edge from one of 256 rows spread over `spread` rad: an error larger
    than e moves a count."""
    g = synthcat.rng_for(96, 71)
    e = synthcat.log_edges(0.02, 60.0, 12)
    c = np.array([0.6, 0.64, np.sqrt(1 - 0.36 - 0.4096)])
    rows = c[None, :] + g.uniform(-spread, spread, size=(256, 3))
    rows /= np.linalg.norm(rows, axis=1)[:, None]
    n = 8192
    a, k, ph = rows[g.integers(0, 256, n)], g.integers(0, e.size, n), g.uniform(0, 2 * np.pi, n)
    th = np.radians(e[k])
    q = 4.0 * np.sin(0.5 * th) ** 2
    r2 = 3.0 * spread ** 2
    err = 2.0 ** -24 * (24.0 * (np.sqrt(q) + np.sqrt(r2)) ** 2 + 640.0 * r2) + 3e-13
    q = np.clip(q + err * g.uniform(-3.0, 3.0, n), 1e-14, 3.9)
    th = 2.0 * np.arcsin(0.5 * np.sqrt(q))
    t1 = np.cross(a, [0.0, 0.0, 1.0])
    t1 /= np.linalg.norm(t1, axis=1)[:, None]
    t2 = np.cross(a, t1)
    cols = np.cos(th)[:, None] * a + np.sin(th)[:, None] * (np.cos(ph)[:, None] * t1 + np.sin(ph)[:, None] * t2)
    cols /= np.linalg.norm(cols, axis=1)[:, None]
    x, y = rows.T.copy(), cols.T.copy()
    ca, cb = ctx.upload_catalog_xyz(*x), ctx.upload_catalog_xyz(*y)
    want = oracle.count(oracle.DR, x, e, b_xyz=y)
    try:
        for per_lane in (2, 4):
            ctx.set_tuning(rows_per_lane=per_lane)
            assert np.array_equal(ctx.count(tp.DR, ca, e, cat_b=cb), want)
            assert np.array_equal(ctx.count(tp.DR, cb, e, cat_b=ca), want)
    finally:
        ctx.set_tuning()
        ctx.release_catalog(ca)
        ctx.release_catalog(cb)
