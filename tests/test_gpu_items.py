"""Work items against the oracle (GPU): cells of few and of many chunks (their
items are emitted by a thread or by a wavefront), items with fewer and more
changed entries than the slab masks start from and than one tile holds, cells
without edges, and moves that leave the grid."""
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


@pytest.mark.parametrize("kind", ["planar", "spatial"])
@pytest.mark.parametrize("cells", [1, 2, 5, 20])
@pytest.mark.parametrize("item_edges", [1, 37, 64, 511])
@pytest.mark.parametrize("n_boxes", [4, 16, 17, 64, 65, 150])
def test_items(ctx, kind, cells, item_edges, n_boxes):
    """n_boxes moved at once: 2 n_boxes changed entries around 32, 33, 128 and
    300; a cell then holds from one item to some thousand."""
    from paper_2603_28674_amd import rgg
    import oracle
    if kind == "planar":
        w = synth.planar_rigid(seed=n_boxes, n_nodes=500, n_boxes=n_boxes, n_updates=2, n_move=n_boxes, world=30.0,
                               resolution=0.5)
        world = 30.0
    else:
        w = synth.spatial_rigid(seed=n_boxes, n_nodes=400, n_boxes=n_boxes, n_updates=2, move_frac=1.0, world=3.0,
                                samples=5)
        world = 3.0
    out = w.boxes[-1].copy()          # half of the boxes leave the grid, then come back
    out[::2, :2] += 50.0 * world
    out[::2, 3:5] += 50.0 * world
    w.boxes = w.boxes + [out, w.boxes[-1]]
    rng = np.random.default_rng(cells)
    for prec in (rgg.RGG_PREC_FP64, rgg.RGG_PREC_FP32_RECHECK):
        g = rgg.Roadmap.from_workload(ctx, w, precision=prec, cell_size=-1.0 if cells == 1 else world / cells,
                                      item_edges=item_edges)
        o = oracle.from_workload(w)
        prev = w.absent()
        for cur in w.boxes:
            ol, og = o.update(prev, cur)
            gl, gg, n, _ = g.update(prev, cur)
            assert np.array_equal(gl, ol) and np.array_equal(gg, og)
            prev = cur
        g.close()


@pytest.mark.parametrize("mode", [{}, {"outer_obb": True}, {"inner_splines": True},
                                  {"outer_obb": True, "inner_splines": True}])
@pytest.mark.parametrize("kind", ["planar", "spatial"])
@pytest.mark.parametrize("items", [1, 767, 768, 769, 1600])
def test_item_counts(ctx, kind, mode, items):
    """One cell of 1 to 1,600 items, around the count up to which three blocks
    share a CU."""
    from paper_2603_28674_amd import rgg
    import oracle
    n, chunk = (400, 511) if items == 1 else (items, 1)
    if kind == "planar":
        w = synth.planar_rigid(seed=7, n_nodes=500, n_boxes=40, n_updates=2, n_move=20, world=30.0, resolution=0.5)
    else:
        w = synth.spatial_rigid(seed=7, n_nodes=500, n_boxes=40, n_updates=2, move_frac=0.5, world=3.0, samples=5)
    assert w.n_edges >= n
    w.edges = w.edges[:n]
    g = rgg.Roadmap.from_workload(ctx, w, precision=rgg.RGG_PREC_FP32_RECHECK, cell_size=-1.0, item_edges=chunk, **mode)
    o = oracle.from_workload(w, **mode)
    prev = w.absent()
    for cur in w.boxes:
        ol, og = o.update(prev, cur)
        gl, gg, _, _ = g.update(prev, cur)
        assert np.array_equal(gl, ol) and np.array_equal(gg, og)
        prev = cur
    g.close()
