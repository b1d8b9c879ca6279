"""Page-locked host memory of the host-buffer update (GPU): more than 64 KB are
held from the second call that asks for an output, never by a roadmap updated
otherwise, and done without where there is none.  Every output is the oracle's."""
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


def workload(n_nodes=1600):
    return synth.planar_rigid(seed=9, n_nodes=n_nodes, n_boxes=40, n_updates=4, resolution=0.5)


def held(E):
    return (E + 255) // 256 * 256 + 8 * E


def test_held_from_the_second_use(ctx):
    import torch
    from paper_2603_28674_amd import rgg
    w = workload()
    E = w.n_edges
    assert held(E) > 65536
    g = rgg.Roadmap.from_workload(ctx, w, precision=1)
    assert rgg.rgg_debug_pinned(g.h) == 0
    # updates that name no host output hold none: device buffers, then nothing asked for
    states = torch.from_numpy(np.stack([w.absent()] + w.boxes)).cuda()
    lab, gray = torch.zeros(E, dtype=torch.uint8, device="cuda"), torch.zeros(E, dtype=torch.int64, device="cuda")
    res = torch.zeros(rgg.RESULT_BYTES, dtype=torch.uint8, device="cuda")
    g.update_async(torch.cuda.current_stream().cuda_stream, states[0], states[1], lab, gray, res)
    g.update(w.boxes[0], w.boxes[1], want_labels=False, gray_cap=0)
    assert rgg.rgg_debug_pinned(g.h) == 0
    for prev, cur, kw, n in ((1, 2, dict(want_labels=True, gray_cap=0), 0), (2, 3, dict(), held(E)), (3, 1, dict(), held(E))):
        g.update(w.boxes[prev], w.boxes[cur], **kw)
        assert rgg.rgg_debug_pinned(g.h) == n
    g.close()


@pytest.mark.parametrize("short", [True, False])
def test_outputs_without_room(ctx, short):
    from paper_2603_28674_amd import rgg
    import oracle
    w = workload()
    E = w.n_edges
    g, o = rgg.Roadmap.from_workload(ctx, w, precision=1), oracle.from_workload(w)
    rgg.rgg_debug_pinned(g.h, held(E) - int(short))
    prev = w.absent()
    for u, cur in enumerate(w.boxes):
        ol, og = o.update(prev, cur)
        cap = 5 if u == 1 else E
        gl, gg, n, r = g.update(prev, cur, want_labels=u != 0, gray_cap=cap)
        assert np.array_equal(gg, og[:cap]) and n == r.n_gray == len(og) > 5
        assert u == 0 or np.array_equal(gl, ol)
        prev = cur
    assert rgg.rgg_debug_pinned(g.h, -1) == (0 if short else held(E))
    # a stale state changes nothing; without the limit the outputs stay the oracle's
    with pytest.raises(rgg.RggError):
        g.update(w.boxes[0], w.boxes[0])
    ol, og = o.update(prev, w.boxes[1])
    gl, gg, n, r = g.update(prev, w.boxes[1])
    assert np.array_equal(gl, ol) and np.array_equal(gg, og) and rgg.rgg_debug_pinned(g.h) == held(E)
    g.close()


@pytest.mark.parametrize("n_nodes", [12, 300, 1240, 1280])   # below 64 KB, and around it
def test_small_outputs(ctx, n_nodes):
    from paper_2603_28674_amd import rgg
    import oracle
    w = workload(n_nodes)
    g, o = rgg.Roadmap.from_workload(ctx, w, precision=1), oracle.from_workload(w)
    assert rgg.rgg_debug_pinned(g.h) == (held(w.n_edges) if held(w.n_edges) <= 65536 else 0)
    prev = w.absent()
    for cur in w.boxes:
        ol, og = o.update(prev, cur)
        gl, gg, n, r = g.update(prev, cur)
        assert np.array_equal(gl, ol) and np.array_equal(gg, og) and n == r.n_gray
        prev = cur
    assert rgg.rgg_debug_pinned(g.h) == held(w.n_edges)
    g.close()
