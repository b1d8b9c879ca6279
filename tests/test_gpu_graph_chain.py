"""Graphs of several updates of one roadmap (GPU): chains launched as kernels (up
to nine) and captured ones, each relaunched from alternating streams with eager
updates between, every output of every launch the oracle's."""
import numpy as np
import pytest

from paper_2603_28674_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2603_28674_amd import rgg
    c = rgg.rgg_context_create(0)
    yield c
    rgg.rgg_context_destroy(c)


# updates of three kernels, and of four (every pair listed)
@pytest.mark.parametrize("n,listing", [(1, False), (2, False), (3, False), (4, False), (7, False), (2, True), (3, True)])
def test_graph_of_several_updates(ctx, n, listing):
    import torch
    from paper_2603_28674_amd import rgg
    import oracle
    w = synth.spatial_rigid(seed=40 + n, n_nodes=1500, n_boxes=60, n_updates=n, world=4.0)
    g = rgg.Roadmap.from_workload(ctx, w, precision=rgg.RGG_PREC_FP32_RECHECK,
                                  **(dict(inline_rounds=rgg.RGG_INLINE_NONE) if listing else {}))
    boxes = w.boxes[:n + 1]                      # the graph goes from state 0 to state n
    states = torch.from_numpy(np.stack(boxes)).cuda()
    first = torch.from_numpy(w.absent()).cuda()
    o = oracle.from_workload(w)
    want = [o.update(w.absent(), boxes[0])] + [o.update(boxes[u], boxes[u + 1]) for u in range(n)]

    def buffers():
        return (torch.zeros(w.n_edges, dtype=torch.uint8, device="cuda"),
                torch.zeros(w.n_edges, dtype=torch.int64, device="cuda"),
                torch.zeros(rgg.RESULT_BYTES, dtype=torch.uint8, device="cuda"))

    outs = [buffers() for _ in range(n + 1)]     # outs[u]: the outputs at state u
    graph = rgg.rgg_graph_create(ctx, [
        rgg.rgg_update_req(g.h.value, w.n_slots, states[u].data_ptr(), states[u + 1].data_ptr(), outs[u + 1][0].data_ptr(),
                           outs[u + 1][1].data_ptr(), w.n_edges, outs[u + 1][2].data_ptr()) for u in range(n)])
    streams = [torch.cuda.Stream() for _ in range(3)]
    at = first
    for rep in range(4):
        for buf in outs:
            for t in buf:
                t.zero_()
        torch.cuda.synchronize()
        # back to state 0 and through the graph, on two streams with nothing
        # waited for between them
        g.update_async(streams[rep % 3].cuda_stream, at, states[0], *outs[0])
        rgg.rgg_graph_launch(graph, streams[(rep + 1) % 3].cuda_stream)
        torch.cuda.synchronize()
        for u in range(n + 1):
            lab, gray, res = outs[u]
            r = rgg.result_from_tensor(res)
            ol, og = want[u]
            assert r.status == 0 and r.n_gray == len(og)
            assert np.array_equal(lab.cpu().numpy(), ol) and np.array_equal(gray[:r.n_gray].cpu().numpy(), og)
        at = states[n]
    rgg.rgg_graph_destroy(graph)
    g.close()
