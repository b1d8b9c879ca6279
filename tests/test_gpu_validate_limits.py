"""Full validation at the limits of a block's LDS (GPU): robots of 64 spheres, in
3-D and on 32 links, with as many slots as are kept in LDS and one more, and
512 active intervals: from 68 to 71 KB of LDS a block, or the boxes left in memory.
Verdicts, levels and witnesses are the oracle's, bit for bit."""
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


def workload(kind, n_boxes):
    rng = np.random.default_rng(n_boxes)
    if kind == "spatial":
        w = synth.spatial_rigid(seed=n_boxes, n_nodes=200, n_boxes=n_boxes, n_updates=0, world=1.5, samples=3)
        w.robot = dataclasses.replace(w.robot, sphere_pos=rng.uniform(-0.5, 0.5, (64, 3)),
                                      sphere_radius=rng.uniform(0.02, 0.08, 64))
        w.boxes = [synth.random_boxes(rng, n_boxes, 3, 0.005, 0.03, -0.5, 2.0)]
    else:
        w = synth.planar_arm(seed=n_boxes, n_nodes=200, n_boxes=n_boxes, n_updates=0, samples=3, n_links=32)
        w.robot = dataclasses.replace(w.robot, sphere_pos=w.robot.sphere_pos[:64], sphere_radius=w.robot.sphere_radius[:64],
                                      sphere_link=np.repeat(np.arange(32, dtype=np.int32), 2))
        rho = float(np.sum(w.robot.link_length))
        w.boxes = [synth.random_boxes(rng, n_boxes, 2, 0.005, 0.03, -rho, rho)]
    # 36 boxes: some edges stay free, some are searched deeply
    w.boxes[0][rng.permutation(n_boxes)[36:]] = synth.ABSENT_BOX
    return w


@pytest.mark.parametrize("kind", ["spatial", "arm"])
@pytest.mark.parametrize("n_boxes", [40, 512, 513])
def test_most_spheres(ctx, kind, n_boxes):
    from paper_2603_28674_amd import rgg
    import oracle
    w = workload(kind, n_boxes)
    g = rgg.Roadmap.from_workload(ctx, w, precision=rgg.RGG_PREC_FP32_RECHECK)
    o = oracle.from_workload(w)
    g.update(w.absent(), w.boxes[0])
    o.update(w.absent(), w.boxes[0])
    ids = np.random.default_rng(1).choice(w.n_edges, size=120, replace=False).astype(np.int64)
    seen = set()
    for limits in ({}, dict(max_level=24, max_active=512), dict(max_level=3, max_active=512), dict(max_level=24, max_active=1)):
        got, want = g.validate(ids, **limits), o.validate(ids, **limits)
        for a, b in zip(got, want):
            assert np.array_equal(a, b, equal_nan=True)
        seen |= set(want[0].tolist())
    assert len(seen) >= 2
    g.close()
