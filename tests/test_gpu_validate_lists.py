"""Full validation where its candidate lists change form (GPU): boxes kept in
LDS or scanned in memory (512 slots), a page of staged boxes (64), the list of
candidates (256), candidates dropped between levels (from 16), lists longer
than the grid holds, one sphere, many links.  Verdicts, levels and witnesses
are the oracle's, bit for bit."""
import dataclasses

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


def workload(kind, n_boxes, seed, n_nodes=250):
    """A roadmap in a small world with many small boxes, so that an edge's
    region holds a large part of them."""
    rng = np.random.default_rng(seed)
    if kind == "planar":
        w = synth.planar_rigid(seed=seed, n_nodes=n_nodes, n_boxes=n_boxes, n_updates=0, world=12.0, resolution=0.5)
        w.boxes = [synth.random_boxes(rng, n_boxes, 2, 0.01, 0.05, 0.0, 12.0)]
    elif kind == "spatial":
        w = synth.spatial_rigid(seed=seed, n_nodes=n_nodes, n_boxes=n_boxes, n_updates=0, world=1.5, samples=3)
        w.boxes = [synth.random_boxes(rng, n_boxes, 3, 0.005, 0.03, -0.5, 2.0)]
    else:
        w = synth.planar_arm(seed=seed, n_nodes=n_nodes, n_boxes=n_boxes, n_updates=0, samples=3,
                             n_links=13 if kind == "arm13" else 7)
        rho = float(np.sum(w.robot.link_length))
        w.boxes = [synth.random_boxes(rng, n_boxes, 2, 0.005, 0.03, -rho, rho)]
        if kind == "arm1":   # one sphere, on the last link
            w.robot = dataclasses.replace(w.robot, sphere_pos=w.robot.sphere_pos[-1:],
                                          sphere_radius=w.robot.sphere_radius[-1:], sphere_link=w.robot.sphere_link[-1:])
    # some slots ABSENT: they are never candidates
    w.boxes[0][:: 9] = synth.ABSENT_BOX
    return w


def check(ctx, w, ids, **limits):
    from paper_2603_28674_amd import rgg
    import oracle
    g = rgg.Roadmap.from_workload(ctx, w, precision=rgg.RGG_PREC_FP32_RECHECK)
    o = oracle.from_workload(w)
    g.update(w.absent(), w.boxes[0])
    o.update(w.absent(), w.boxes[0])
    got, want = g.validate(ids, **limits), o.validate(ids, **limits)
    for a, b in zip(got, want):
        assert np.array_equal(a, b, equal_nan=True)
    g.close()
    return want


@pytest.mark.parametrize("kind", ["planar", "spatial", "arm", "arm1", "arm13"])
@pytest.mark.parametrize("n_boxes", [1, 17, 70, 300, 512, 513, 1200])
def test_candidate_lists(ctx, kind, n_boxes):
    w = workload(kind, n_boxes, seed=70 + n_boxes)
    ids = np.random.default_rng(n_boxes).choice(w.n_edges, size=150, replace=False).astype(np.int64)
    check(ctx, w, ids)
    # tight limits: UNRESOLVED at the level and at the active count
    check(ctx, w, ids, max_level=2, max_active=256)
    check(ctx, w, ids, max_level=24, max_active=1)


@pytest.mark.parametrize("n", [1, 3, 4, 5, 2047, 2049, 12000])
def test_list_lengths_and_repeats(ctx, n):
    """Lists shorter than a block, around the grid's first round and well past
    it, with edges named more than once."""
    w = workload("planar", 40, seed=5, n_nodes=900)
    ids = np.random.default_rng(n).integers(0, w.n_edges, size=n).astype(np.int64)
    verdict, _, _ = check(ctx, w, ids)
    assert len(verdict) == n
