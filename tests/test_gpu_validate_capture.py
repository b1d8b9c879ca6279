"""A captured update with its validation, replayed (GPU): every replay's labels,
gray ids, verdicts, levels and witnesses are the oracle's, and nothing is
written past the gray list's end."""
import numpy as np
import pytest

from paper_2603_28674_amd import synth

pytestmark = pytest.mark.gpu

KIND = {"planar": dict(f="planar_rigid", n_nodes=900, n_boxes=40, resolution=0.5),
        "spatial": dict(f="spatial_rigid", n_nodes=2000, n_boxes=80, world=4.0),
        "arm": dict(f="planar_arm", n_nodes=1200, n_boxes=60)}


@pytest.mark.parametrize("kind", sorted(KIND))
def test_captured_validation(kind):
    import torch
    from paper_2603_28674_amd import rgg
    import oracle
    ctx = rgg.rgg_context_create(0)
    kw = dict(KIND[kind])
    w = getattr(synth, kw.pop("f"))(seed=17, n_updates=3, **kw)
    E = w.n_edges
    g = rgg.Roadmap.from_workload(ctx, w, precision=rgg.RGG_PREC_FP32_RECHECK)
    states = [torch.from_numpy(b.copy()).cuda() for b in [w.absent()] + w.boxes]
    old, new = states[0].clone(), states[1].clone()
    lab, ver = (torch.zeros(E, dtype=torch.uint8, device="cuda") for _ in range(2))
    gray, lev = torch.zeros(E, dtype=torch.int64, device="cuda"), torch.zeros(E, dtype=torch.int32, device="cuda")
    wit = torch.zeros(E, dtype=torch.float64, device="cuda")
    res = torch.zeros(rgg.RESULT_BYTES, dtype=torch.uint8, device="cuda")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        s = torch.cuda.current_stream().cuda_stream
        g.update_async(s, old, new, lab, gray, res)
        rgg.rgg_validate_async(g.h, s, gray, E, res, ver, lev, wit)
    o = oracle.from_workload(w)
    for u in range(len(w.boxes)):
        old.copy_(states[u])
        new.copy_(states[u + 1])
        for t, v in ((lab, 99), (ver, 99), (gray, -7), (lev, -7), (wit, -7.0)):
            t.fill_(v)
        graph.replay()
        torch.cuda.synchronize()
        ol, og = o.update(w.boxes[u - 1] if u else w.absent(), w.boxes[u])
        want, n = o.validate(og), len(og)
        assert n > 0 and np.array_equal(lab.cpu().numpy(), ol) and np.array_equal(gray[:n].cpu().numpy(), og)
        for t, x in zip((ver, lev, wit), want):
            assert np.array_equal(t[:n].cpu().numpy(), x, equal_nan=True)
        assert bool((ver[n:] == 99).all()) and bool((lev[n:] == -7).all()) and bool((wit[n:] == -7.0).all())
    g.close()
    rgg.rgg_context_destroy(ctx)
