"""Counts captured into a caller's graph (needs an MI355X): tpcf_count_async on
a borrowed stream that is capturing."""

import ctypes

import numpy as np
import pytest

import oracle
import paper_1204_6630_amd as tp
import synthcat

pytestmark = pytest.mark.gpu


def _kernel_nodes(graph):
    """Kernel nodes of a torch graph kept after its capture; every node is one."""
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    h, n = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(h, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(h, nodes, ctypes.byref(n)) == 0
    for k in nodes:
        kind = ctypes.c_int(-1)
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(k), ctypes.byref(kind)) == 0
        assert kind.value == 0
    return n.value


@pytest.mark.parametrize("prec", [tp.FP32_CHORD, tp.FP64])
def test_captured_counts_clear_their_own_buffers(prec):
    """Each captured count holds the clearing of its histogram copies and
    queues, whatever they held at the capture: a graph does not rely on other
    launches.  Replayed with eager counts of other sizes in between, on the
    same workspace, every result equals the oracle's."""
    import torch
    g = synthcat.rng_for(96, 61)
    fp = (20.0, 30.0, -5.0, 5.0)
    d, r = synthcat.uniform_patch(1500, fp, g), synthcat.uniform_patch(2100, fp, g)
    e, few = synthcat.log_edges(0.05, 9.0, 12), np.array([1.0, 4.0])
    xd, xr = oracle.radec_to_xyz(*d), oracle.radec_to_xyz(*r)
    want = [oracle.count(oracle.DD, xd, e), oracle.count(oracle.DR, xd, e, b_xyz=xr)]
    want_few = oracle.count(oracle.DR, xd, few, b_xyz=xr)
    s = torch.cuda.Stream()
    with tp.Context(0, s.cuda_stream) as ctx, torch.cuda.stream(s):
        a, b = ctx.upload_catalog(*d), ctx.upload_catalog(*r)
        out = torch.zeros((3, e.size + 1), dtype=torch.int64, device="cuda")

        def both():
            ctx.count_async(tp.DD, a, e, out[0].data_ptr(), precision=prec)
            ctx.count_async(tp.DR, a, e, out[1].data_ptr(), cat_b=b, precision=prec)

        def eager():
            ctx.count_async(tp.DR, a, few, out[2].data_ptr(), cat_b=b, precision=prec)

        both()
        eager()
        s.synchronize()
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph, stream=s):
            both()
        assert _kernel_nodes(graph) == 6        # clear, pairs, reduce; twice
        graph.instantiate()
        for k in range(4):
            out.zero_()
            if k % 2:
                eager()
            graph.replay()
            if k > 1:
                eager()
                assert np.array_equal(ctx.count(tp.DD, a, e, precision=prec), want[0])
            s.synchronize()
            got = out.cpu().numpy().view(np.uint64)
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
            if k:
                assert np.array_equal(got[2, :few.size + 1], want_few)
        del graph
        torch.cuda.synchronize()
