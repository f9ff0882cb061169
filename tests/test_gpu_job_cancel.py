"""What being cancellable costs a submitted job, and what a cancellation saves
(needs an MI355X)."""

import time

import numpy as np
import pytest

import paper_1204_6630_amd as tp
import synthcat

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tp.Context(0)
    yield c
    c.close()


def _median_us(f, n=21):
    t = []
    for _ in range(n):
        a = time.perf_counter()
        f()
        t.append(time.perf_counter() - a)
    return 1e6 * float(np.median(t))


@pytest.mark.parametrize("prec", [tp.FP32_CHORD, tp.FP64])
def test_short_job_takes_what_a_count_takes(ctx, prec):
    """The flag of a job that can be cancelled lies in host memory: 2500
    wavefronts that read it take longer than a short job itself."""
    g = synthcat.rng_for(96, 2)
    a = ctx.upload_catalog(*synthcat.uniform_patch(637, synthcat.OCTANT, g))
    b = ctx.upload_catalog(*synthcat.uniform_patch(55_000, synthcat.OCTANT, g))
    e = synthcat.log_edges(0.01, 20.0, 30)
    want = ctx.count(tp.DR, a, e, cat_b=b, precision=prec)

    def job():
        assert np.array_equal(ctx.wait(ctx.submit(tp.DR, a, e, cat_b=b, precision=prec), e.size + 1), want)

    job()
    count = _median_us(lambda: ctx.count(tp.DR, a, e, cat_b=b, precision=prec))
    assert _median_us(job) < 2.0 * count + 20.0
    ctx.release_catalog(a)
    ctx.release_catalog(b)


def test_cancelled_long_job_ends_early(ctx):
    """Every wavefront looks at the flag after its first two million pairs:
    5e11 pairs in FP64, cancelled at once, take a fraction of their time."""
    g = synthcat.rng_for(96, 3)
    big = ctx.upload_catalog(*synthcat.uniform_patch(1_000_000, synthcat.OCTANT, g))
    e = synthcat.log_edges(0.01, 10.0, 20)

    def run(cancel):
        t = time.perf_counter()
        jid = ctx.submit(tp.DD, big, e, precision=tp.FP64)
        if cancel:
            ctx.cancel(jid)
            with pytest.raises(tp.TpcfError) as ei:
                ctx.wait(jid, e.size + 1)
            assert ei.value.code == -6
        else:
            assert int(ctx.wait(jid, e.size + 1).sum()) == 1_000_000 * 999_999 // 2
        return time.perf_counter() - t

    full = run(False)
    assert min(run(True) for _ in range(3)) < 0.5 * full
    ctx.release_catalog(big)
