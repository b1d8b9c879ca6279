"""Label tiles around the number from which the label kernel runs in blocks of
1,024 threads (GPU): whole and ragged tiles on both sides, against the oracle."""
import numpy as np
import pytest

from paper_2603_28674_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def work():
    return synth.planar_rigid(seed=12, n_nodes=9500, n_boxes=30, n_updates=1, resolution=1.0)


@pytest.mark.parametrize("edges", [11 * 4096 - 1, 11 * 4096, 11 * 4096 + 1, 12 * 4096, 12 * 4096 + 3])
def test_label_blocks(work, edges):
    import dataclasses
    from paper_2603_28674_amd import rgg
    import oracle
    assert work.n_edges >= edges
    w = dataclasses.replace(work, edges=work.edges[:edges])
    ctx = rgg.rgg_context_create(0)
    g, o = rgg.Roadmap.from_workload(ctx, w, precision=rgg.RGG_PREC_FP32_RECHECK), oracle.from_workload(w)
    prev = w.absent()
    for cur in w.boxes:
        ol, og = o.update(prev, cur)
        gl, gg, n, r = g.update(prev, cur)
        assert np.array_equal(gl, ol) and np.array_equal(gg, og) and n == r.n_gray == len(og) > 0
        prev = cur
    g.close()
    rgg.rgg_context_destroy(ctx)
