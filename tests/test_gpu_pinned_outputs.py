"""Page-locked host memory of the host-buffer update (GPU): held from the first
call that asks for an output, never by a roadmap updated otherwise, and done
without where there is none.  Every output is the oracle's."""
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


def workload():
    return synth.planar_rigid(seed=9, n_nodes=1200, n_boxes=40, n_updates=4, resolution=0.5)


def test_held_from_the_first_use(ctx):
    import torch
    from paper_2603_28674_amd import rgg
    w = workload()
    E = w.n_edges
    g = rgg.Roadmap.from_workload(ctx, w, precision=1)
    assert rgg.rgg_debug_pinned(g.h) == 0
    # updates that name no host output hold none: device buffers, then nothing asked for
    states = torch.from_numpy(np.stack([w.absent()] + w.boxes)).cuda()
    lab, gray = torch.zeros(E, dtype=torch.uint8, device="cuda"), torch.zeros(E, dtype=torch.int64, device="cuda")
    res = torch.zeros(rgg.RESULT_BYTES, dtype=torch.uint8, device="cuda")
    g.update_async(torch.cuda.current_stream().cuda_stream, states[0], states[1], lab, gray, res)
    g.update(w.boxes[0], w.boxes[1], want_labels=False, gray_cap=0)
    assert rgg.rgg_debug_pinned(g.h) == 0
    g.update(w.boxes[1], w.boxes[2], want_labels=True, gray_cap=0)
    assert rgg.rgg_debug_pinned(g.h) == E
    for prev, cur in ((2, 3), (3, 1)):
        g.update(w.boxes[prev], w.boxes[cur])
        assert rgg.rgg_debug_pinned(g.h) == 9 * E
    g.close()


@pytest.mark.parametrize("room", ["none", "labels", "ids", "both"])
def test_outputs_without_room(ctx, room):
    from paper_2603_28674_amd import rgg
    import oracle
    w = workload()
    E = w.n_edges
    g, o = rgg.Roadmap.from_workload(ctx, w, precision=1), oracle.from_workload(w)
    limit = {"none": 0, "labels": E, "ids": 8 * E, "both": 9 * E}[room]
    rgg.rgg_debug_pinned(g.h, limit)
    prev = w.absent()
    for u, cur in enumerate(w.boxes):
        ol, og = o.update(prev, cur)
        cap = 5 if u == 1 else E
        gl, gg, n, r = g.update(prev, cur, want_labels=u != 0, gray_cap=cap)   # ids alone first
        assert np.array_equal(gg, og[:cap]) and n == r.n_gray == len(og) > 5
        assert u == 0 or np.array_equal(gl, ol)
        assert rgg.rgg_debug_pinned(g.h, limit) <= limit
        prev = cur
    held = rgg.rgg_debug_pinned(g.h, -1)
    assert held == {"none": 0, "labels": E, "ids": 8 * E, "both": 9 * E}[room]
    # a stale state changes nothing; without the limit the rest is held and the outputs stay the oracle's
    with pytest.raises(rgg.RggError):
        g.update(w.boxes[0], w.boxes[0])
    ol, og = o.update(prev, w.boxes[1])
    gl, gg, n, r = g.update(prev, w.boxes[1])
    assert np.array_equal(gl, ol) and np.array_equal(gg, og) and rgg.rgg_debug_pinned(g.h) == 9 * E
    g.close()
