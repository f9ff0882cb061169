"""Requests of a few rows against many columns (needs an MI355X): tiles that
are nearly empty, cut into as many units as full ones would be."""

import ctypes

import numpy as np
import pytest

import paper_1204_6630_amd as tp
import synthcat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 3])
def test_noalloc_of_few_rows_and_many_columns(rows):
    """25 million columns in chunks of 64 are more units than the fixed work
    area holds: the chunks widen, and the counts equal tpcf_count's."""
    import torch
    n = 25_000_000
    g = torch.Generator(device="cuda").manual_seed(7)
    v = torch.randn((3, n), dtype=torch.float64, device="cuda", generator=g)
    v /= torch.linalg.norm(v, dim=0)
    torch.cuda.synchronize()
    e = np.ascontiguousarray(synthcat.log_edges(0.01, 60.0, 20))
    with tp.Context(0) as ctx:
        c = ctx.attach_catalog(v)
        for prec in (tp.FP32_CHORD, tp.FP64):
            out = np.zeros(e.size + 1, dtype=np.uint64)
            rc = tp.lib().tpcf_count_noalloc(ctx.handle, tp.DR, c, c, e.ctypes.data, e.size - 1, prec, 5, 5 + rows,
                                             out.ctypes.data)
            assert rc == 0, ctypes.string_at(tp.lib().tpcf_last_error(None))
            assert int(out.sum()) == rows * n
            assert np.array_equal(out, ctx.count(tp.DR, c, e, cat_b=c, precision=prec, row_begin=5, row_end=5 + rows))
