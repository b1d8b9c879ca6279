"""The quick capsule tests of the item kernels against the oracle (GPU), where
their margins matter: boxes tangent to end copies and capsule ends within
1e-17 to 1e-9 of the radius, exactly tangent ones (one sphere sliding along a
face on exact binary coordinates), one to 64 spheres per robot, and more open
capsule tests than their queue holds."""
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


def check(ctx, w, precision, **kw):
    from paper_2603_28674_amd import rgg
    import oracle
    g = rgg.Roadmap.from_workload(ctx, w, precision=precision, **kw)
    o = oracle.from_workload(w, outer_obb=kw.get("outer_obb", False), inner_splines=kw.get("inner_splines", False))
    prev, mix = w.absent(), np.zeros(3, dtype=int)
    for cur in w.boxes:
        ol, og = o.update(prev, cur)
        gl, gg, n, _ = g.update(prev, cur)
        assert np.array_equal(gl, ol) and np.array_equal(gg, og) and n == len(og)
        mix += np.bincount(ol, minlength=3)
        prev = cur
    g.close()
    return mix


def end_tangent_boxes(w, rng, n, which):
    """Boxes whose one face is at r (1 +- eps) from the first or last copy of a
    random edge's sphere (which = "copy"), or at R (1 +- eps) from an end of
    its capsule ("capsule")."""
    import oracle
    o = oracle.from_workload(w)
    D, B = w.robot.dim, w.robot.n_spheres
    out = np.tile(synth.ABSENT_BOX, (n, 1))
    for k in range(n):
        e, i = int(rng.integers(w.n_edges)), int(rng.integers(B))
        A = o.centres(e)[0 if rng.random() < 0.5 else -1, i]
        rad = w.robot.sphere_radius[i] if which == "copy" else o.capsule_radius(e)[i]
        d = int(rng.integers(D))
        sgn = 1.0 if rng.random() < 0.5 else -1.0
        eps = (0.0 if rng.random() < 0.2 else 10.0 ** rng.uniform(-17, -9)) * (1 if rng.random() < 0.5 else -1)
        lo, hi = np.zeros(3), np.zeros(3)
        lo[:D], hi[:D] = A - 0.3, A + 0.3
        face = A[d] + sgn * rad * (1.0 + eps)
        if sgn > 0:
            lo[d], hi[d] = face, face + 0.5
        else:
            lo[d], hi[d] = face - 0.5, face
        out[k, :3], out[k, 3:] = lo, hi
    return out


@pytest.mark.parametrize("kind", ["planar", "spatial", "arm"])
@pytest.mark.parametrize("which", ["copy", "capsule"])
@pytest.mark.parametrize("mode", [{}, {"outer_obb": True}])
def test_tangent_to_the_ends(ctx, kind, which, mode):
    from paper_2603_28674_amd import rgg
    make = {"planar": lambda: synth.planar_rigid(seed=3, n_nodes=400, n_boxes=60, n_updates=0),
            "spatial": lambda: synth.spatial_rigid(seed=4, n_nodes=400, n_boxes=60, n_updates=0, world=5.0),
            "arm": lambda: synth.planar_arm(seed=5, n_nodes=300, n_boxes=12, n_updates=0)}[kind]
    w = make()
    rng = np.random.default_rng(len(kind) + len(which))
    n = w.n_slots
    w.boxes = [end_tangent_boxes(w, rng, n, which), end_tangent_boxes(w, rng, n, which)]
    for prec in (rgg.RGG_PREC_FP64, rgg.RGG_PREC_FP32_RECHECK):
        check(ctx, w, prec, **mode)


@pytest.mark.parametrize("precision", [0, 1])
def test_exact_ties(ctx, precision):
    """Discs of exact binary radius translating along faces at exactly that
    distance (closed sets: they touch), and one ulp nearer and farther."""
    n = 64
    x = np.arange(n) * 0.25
    q = np.stack([x, np.full(n, 2.0), np.zeros(n)], axis=1)
    edges = np.stack([np.arange(n - 1), np.arange(1, n)], axis=1).astype(np.int64)
    robot = synth.Robot(synth.SE2, np.array([[0.0, 0.0], [0.0, 0.5]]), np.array([0.25, 0.5]))
    top = [1.75, np.nextafter(1.75, 0), np.nextafter(1.75, 2), 1.5]
    boxes = []
    for t in top:
        b = np.zeros((2, 6))
        b[0] = [3.0, 0.0, 0.0, 6.0, t, 0.0]
        b[1] = [9.0, 5.0 - t + 0.25, 0.0, 11.0, 6.0, 0.0]   # above the second disc
        boxes.append(b)
    w = synth.Workload("ties", robot, q, edges, 0.05, 0, boxes, np.zeros(3), np.zeros(3))
    mix = check(ctx, w, precision)
    assert mix[0] > 0 and mix[2] > 0


@pytest.mark.parametrize("B", [1, 2, 3, 31, 33, 63, 64])
@pytest.mark.parametrize("kind", ["se2", "se3"])
@pytest.mark.parametrize("precision", [0, 1])
def test_sphere_counts(ctx, B, kind, precision):
    """Every way a wavefront's lanes split over pairs; long edges among few
    boxes leave most capsule tests open, more than their queue holds at the
    larger counts."""
    rng = np.random.default_rng(B)
    if kind == "se2":
        w = synth.planar_rigid(seed=B, n_nodes=150, n_boxes=30, n_updates=2, world=20.0, resolution=0.5)
        robot = synth.robot_se2(rng, B)
    else:
        w = synth.spatial_rigid(seed=B, n_nodes=150, n_boxes=30, n_updates=2, world=3.0, samples=7)
        robot = synth.robot_se3(rng, B)
    w = dataclasses.replace(w, robot=dataclasses.replace(robot, sphere_radius=robot.sphere_radius * 0.2))
    check(ctx, w, precision)


@pytest.mark.parametrize("kind", ["planar", "spatial"])
@pytest.mark.parametrize("cell_size", [-1.0, 0.0])
@pytest.mark.parametrize("item_edges", [0, 512])
def test_retest_queue_fills(ctx, kind, cell_size, item_edges):
    """Every pair re-tested in binary64, with several tiles of changed entries
    per item, whatever number of pairs a block collects first: labels, pair
    counts and candidate counts do not depend on it."""
    from paper_2603_28674_amd import rgg
    import oracle
    if kind == "planar":
        w = synth.planar_rigid(seed=8, n_nodes=900, n_boxes=180, n_updates=2, n_move=170, world=40.0)
    else:
        w = synth.spatial_rigid(seed=9, n_nodes=900, n_boxes=180, n_updates=2, move_frac=0.9, world=4.0)
    seen = []
    for cap in (1, 5, 64, 0):
        g = rgg.Roadmap.from_workload(ctx, w, precision=rgg.RGG_PREC_FP32_RECHECK, band_rel=float("inf"),
                                      cell_size=cell_size, item_edges=item_edges, retest_capacity=cap)
        o = oracle.from_workload(w)
        prev, counts = w.absent(), []
        for cur in w.boxes:
            ol, og = o.update(prev, cur)
            gl, gg, n, r = g.update(prev, cur)
            assert np.array_equal(gl, ol) and np.array_equal(gg, og)
            assert r.n_rechecked == r.n_pairs > 0
            counts.append((r.n_pairs, r.n_outer_hits, r.n_candidate_edges, r.n_cells_visited))
            prev = cur
        seen.append(counts)
        g.close()
    assert all(x == seen[0] for x in seen)
