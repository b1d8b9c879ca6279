"""Ordering of a roadmap's updates across streams, entry points and captures
(GPU): nothing is waited for between the calls, every result is the oracle's."""
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


class Case:
    def __init__(self, ctx, n_updates, seed=61, precision=1):
        import torch
        from paper_2603_28674_amd import rgg
        import oracle
        w = synth.spatial_rigid(seed=seed, n_nodes=4000, n_boxes=80, n_updates=n_updates, world=5.0)
        self.w = w
        self.g = rgg.Roadmap.from_workload(ctx, w, precision=precision)
        dev = torch.device("cuda:0")
        self.states = [torch.from_numpy(b.copy()).to(dev) for b in [w.absent()] + w.boxes]
        self.labels = torch.zeros(w.n_edges, dtype=torch.uint8, device=dev)
        self.gray = torch.zeros(w.n_edges, dtype=torch.int64, device=dev)
        self.res = torch.zeros(rgg.RESULT_BYTES, dtype=torch.uint8, device=dev)
        o, prev = oracle.from_workload(w), w.absent()
        self.want = []
        for cur in w.boxes:
            self.want.append(o.update(prev, cur))
            prev = cur

    def req(self, u):
        from paper_2603_28674_amd import rgg
        return rgg.rgg_update_req(self.g.h.value, self.w.n_slots, self.states[u].data_ptr(),
                                  self.states[u + 1].data_ptr(), self.labels.data_ptr(), self.gray.data_ptr(),
                                  self.w.n_edges, self.res.data_ptr())

    def check(self, u):
        from paper_2603_28674_amd import rgg
        r = rgg.result_from_tensor(self.res)
        lab, gray = self.want[u]
        assert r.status == 0 and r.n_gray == len(gray)
        assert np.array_equal(self.labels.cpu().numpy(), lab)
        assert np.array_equal(self.gray[: r.n_gray].cpu().numpy(), gray)


@pytest.mark.parametrize("precision", [0, 1])
def test_updates_alternate_streams_and_entry_points(ctx, precision):
    """Update, graph, batch and batch graph on three streams in turn, each
    behind the one before only by the library's own ordering."""
    import torch
    from paper_2603_28674_amd import rgg
    n = 12
    c = Case(ctx, n - 1, precision=precision)
    batch = rgg.rgg_batch_create(ctx, [c.g.h])
    graphs = {u: rgg.rgg_graph_create(ctx, [c.req(u)]) for u in range(1, n, 4)}
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    for u in range(n):
        s = streams[u % 3].cuda_stream
        if u % 4 == 0:
            c.g.update_async(s, c.states[u], c.states[u + 1], c.labels, c.gray, c.res)
        elif u % 4 == 1:
            rgg.rgg_graph_launch(graphs[u], s)
        elif u % 4 == 2:
            rgg.rgg_batch_launch(batch, [c.req(u)], s)
        else:
            rgg.rgg_batch_launch_graph(batch, [c.req(u)], s)
    torch.cuda.synchronize()
    c.check(n - 1)
    # a host-buffer query queued behind the last update, on the roadmap's own stream
    assert np.array_equal(c.g.labels(), c.want[n - 1][0])
    for g in graphs.values():
        rgg.rgg_graph_destroy(g)
    rgg.rgg_batch_destroy(batch)
    c.g.close()


def test_update_then_validation_on_another_stream(ctx):
    """The validation of one stream reads the gray list and the slots that
    the update of another stream wrote."""
    import torch
    from paper_2603_28674_amd import rgg
    c = Case(ctx, 5)
    dev = torch.device("cuda:0")
    ver = torch.zeros(c.w.n_edges, dtype=torch.uint8, device=dev)
    lev = torch.zeros(c.w.n_edges, dtype=torch.int32, device=dev)
    wit = torch.zeros(c.w.n_edges, dtype=torch.float64, device=dev)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for u in range(6):
        c.g.update_async(a.cuda_stream, c.states[u], c.states[u + 1], c.labels, c.gray, c.res)
        rgg.rgg_validate_async(c.g.h, b.cuda_stream, c.gray, c.w.n_edges, c.res, ver, lev, wit)
    torch.cuda.synchronize()
    c.check(5)
    want = c.g.validate(c.want[5][1])
    n = len(c.want[5][1])
    assert n > 0
    assert np.array_equal(ver[:n].cpu().numpy(), want[0]) and np.array_equal(lev[:n].cpu().numpy(), want[1])
    assert np.array_equal(wit[:n].cpu().numpy(), want[2], equal_nan=True)
    c.g.close()


def test_update_and_validation_under_capture(ctx):
    """The caller's own capture of an update and its validation, replayed on a
    round trip of states (the graph's pointers are fixed: the states are
    copied into its two box buffers), every replay checked."""
    import torch
    from paper_2603_28674_amd import rgg
    c = Case(ctx, 3)
    ver = torch.zeros(c.w.n_edges, dtype=torch.uint8, device="cuda")
    lev = torch.zeros(c.w.n_edges, dtype=torch.int32, device="cuda")
    wit = torch.zeros(c.w.n_edges, dtype=torch.float64, device="cuda")
    old, new = c.states[0].clone(), c.states[1].clone()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        s = torch.cuda.current_stream().cuda_stream
        c.g.update_async(s, old, new, c.labels, c.gray, c.res)
        rgg.rgg_validate_async(c.g.h, s, c.gray, c.w.n_edges, c.res, ver, lev, wit)
    for u in range(4):
        old.copy_(c.states[u])
        new.copy_(c.states[u + 1])
        graph.replay()
        torch.cuda.synchronize()
        c.check(u)
