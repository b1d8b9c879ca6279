"""The host-buffer update (GPU): boxes read from pinned memory or copied up
(1,024 slots), outputs asked for or not, the gray list's capacity, no slots and
no edges.  Every output is the oracle's, or untouched."""
import ctypes as C

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


@pytest.mark.parametrize("n_boxes", [1, 511, 512, 513, 1024, 1025, 4096])
def test_slots(ctx, n_boxes):
    from paper_2603_28674_amd import rgg
    import oracle
    w = synth.planar_rigid(seed=n_boxes, n_nodes=700, n_boxes=n_boxes, n_updates=3, n_move=max(1, n_boxes // 8),
                           world=60.0, resolution=0.5)
    g, o = rgg.Roadmap.from_workload(ctx, w, precision=1), oracle.from_workload(w)
    prev = w.absent()
    for cur in w.boxes:
        ol, og = o.update(prev, cur)
        gl, gg, n, r = g.update(prev, cur)
        assert np.array_equal(gl, ol) and np.array_equal(gg, og) and n == r.n_gray == len(og)
        assert np.array_equal(g.labels(), ol)
        prev = cur
    g.close()


def test_outputs(ctx):
    from paper_2603_28674_amd import rgg
    import oracle
    w = synth.planar_rigid(seed=3, n_nodes=1200, n_boxes=40, n_updates=4, resolution=0.5)
    g, o = rgg.Roadmap.from_workload(ctx, w, precision=1), oracle.from_workload(w)
    E, prev = w.n_edges, w.absent()
    for u, cur in enumerate(w.boxes):
        ol, og = o.update(prev, cur)
        assert len(og) > 8
        labels = np.full(E, 77, dtype=np.uint8) if u != 1 else None
        cap = [E, 5, 0, len(og), E + 100][u]
        gray = np.full(E + 100, -7, dtype=np.int64) if u != 2 else None
        n, res = C.c_int64(-1), rgg.rgg_update_result()
        a, b = rgg.boxes_array(prev), rgg.boxes_array(cur)
        st = rgg.lib().rgg_update(g.h, a.shape[0], rgg._ptr(a), rgg._ptr(b), rgg._ptr(labels), rgg._ptr(gray), cap,
                                  C.byref(n), C.byref(res))
        assert st == (rgg.RGG_E_CAPACITY if u == 1 else rgg.RGG_OK) and n.value == res.n_gray == len(og)
        if labels is not None:
            assert np.array_equal(labels, ol)
        if gray is not None:
            k = min(cap, len(og))
            assert np.array_equal(gray[:k], og[:k]) and np.all(gray[k:] == -7)
        prev = cur
    # a stale state changes nothing and writes nothing
    labels, gray = np.full(E, 77, dtype=np.uint8), np.full(E, -7, dtype=np.int64)
    a = rgg.boxes_array(w.boxes[0])
    st = rgg.lib().rgg_update(g.h, a.shape[0], rgg._ptr(a), rgg._ptr(a), rgg._ptr(labels), rgg._ptr(gray), E, None, None)
    assert st == rgg.RGG_E_STATE_MISMATCH and np.all(labels == 77) and np.all(gray == -7)
    assert np.array_equal(g.labels(), ol)
    g.close()


def test_no_slots_and_no_edges(ctx):
    from paper_2603_28674_amd import rgg
    w = synth.planar_rigid(seed=4, n_nodes=100, n_boxes=5, n_updates=0, resolution=0.5)
    g = rgg.Roadmap(ctx, w.robot, w.q, w.edges, 0, resolution=0.5, precision=1)
    lab, gray, n, r = g.update(np.zeros((0, 6)), np.zeros((0, 6)))
    assert not lab.any() and n == 0 and r.status == 0
    g.close()
    g = rgg.Roadmap(ctx, w.robot, w.q, np.zeros((0, 2), dtype=np.int64), 5, resolution=0.5, precision=1)
    lab, gray, n, r = g.update(w.absent(), w.boxes[0])
    assert lab.size == 0 and n == 0 and r.status == 0
    g.close()
