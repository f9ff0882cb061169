"""A batch with more job shapes than the library keeps plans for (needs an
MI355X): every job's counts equal the oracle's."""

import numpy as np
import pytest

import oracle
import paper_1204_6630_amd as tp
import synthcat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("njobs", [255, 256, 300])
def test_more_shapes_than_plans(njobs):
    g = synthcat.rng_for(99, 31)
    e = synthcat.log_edges(0.1, 9.0, 7)
    ctx = tp.Context(0)
    try:
        pts = [synthcat.uniform_patch(n, (20.0, 30.0, -5.0, 5.0), g) for n in range(2, njobs + 2)]
        cats = [ctx.upload_catalog(*p) for p in pts]
        for graph in (False, True):
            got = ctx.count_batch([(tp.DD, c, -1) for c in cats], e, graph=graph)
            for p, h in zip(pts[::29], got[::29]):
                assert np.array_equal(h, oracle.count(oracle.DD, oracle.radec_to_xyz(*p), e))
            for k, p in enumerate(pts):
                n = p[0].size
                assert int(got[k].sum()) == n * (n - 1) // 2
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", [tp.FP32_CHORD, tp.FP64])
@pytest.mark.parametrize("graph", [False, True])
def test_batch_of_empty_requests(graph, prec):
    """No request of the batch has a pair: a catalog of one point, an empty
    one, an empty row range; then the same with one that has."""
    e = np.array([1.0, 5.0])
    ctx = tp.Context(0)
    try:
        one, none, two = (ctx.upload_catalog(*np.full((2, n), 20.0)) for n in (1, 0, 2))
        empty = [(tp.DD, one, -1), (tp.DD, none, -1), (tp.DR, two, none), (tp.DR, none, one), (tp.RR, two, -1, 1, 1)]
        for _ in range(2):
            assert not ctx.count_batch(empty, e, precision=prec, graph=graph).any()
            got = ctx.count_batch(empty + [(tp.DD, two, -1)], e, precision=prec, graph=graph)
            assert not got[:-1].any() and list(got[-1]) == [1, 0, 0]
    finally:
        ctx.close()
