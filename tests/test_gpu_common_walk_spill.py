"""The common walk of the 4-wide traversal with more deferred children than the
16 stack entries held in LDS: pushes and pops of the spill area, and the
hand-over to the per-lane loop with entries there, against testing every
triangle."""
import numpy as np
import pytest

import scenegen as sg
from gpu_helpers import gpu_radio_map

pytestmark = pytest.mark.gpu

STACK_LDS = 16
EMPTY = 0x7fffffff


def _mesh(V):
    n = len(V)
    return sg.Scene(V.reshape(-1, 3).astype(np.float32), np.arange(3 * n, dtype=np.int32).reshape(n, 3),
                    np.zeros(n, np.int32), np.array([5.24]), np.array([0.12]), "slivers")


def _scene(kind):
    """Scenes of more than 4096 triangles (smaller ones have a shallower tree) whose
    boxes are large and seldom hit, so that children stay deferred.  Counted with a
    counter in the kernel, 4,099 rays push 226 k entries to the spill area in
    `slivers` and 1e5 rays 2.9 M in `nested`, where two wavefronts also
    hand over to the per-lane loop with entries there."""
    rng = np.random.default_rng(1)
    if kind == "slivers":                  # thin triangles through the whole volume
        n = 20_000
        c, s = rng.uniform(-5.0, 5.0, (n, 1, 3)), np.exp(rng.uniform(np.log(20.0), np.log(60.0), (n, 1, 1)))
        d = rng.normal(size=(n, 1, 3))
        d /= np.linalg.norm(d, axis=2, keepdims=True)
        e = rng.normal(size=(n, 1, 3)) * 0.01
        return _mesh(np.concatenate([c - d * s, c + d * s, c + d * s * 0.9 + e], 1))
    # thin triangles around a corner at three scales, their boxes all over it, and
    # at the corner small triangles among which the lanes part
    T = []
    for i in range(3):
        c = 100.0 * 2.0 ** -i * rng.uniform(0.5, 1.0, (200, 1, 3)) * (rng.uniform(size=(200, 1, 3)) < 0.6)
        d = rng.choice([-1.0, 1.0], (200, 1, 3)) * rng.uniform(0.8, 1.2, (200, 1, 3)) * 200.0
        T.append(np.concatenate([c - d, c + d, c + d * 0.9 + rng.normal(size=(200, 1, 3)) * 0.01], 1))
    c = rng.uniform(0, 12.5, (60_000, 1, 3))
    T.append(c + rng.normal(size=(60_000, 3, 3)) * 0.03)
    return _mesh(np.concatenate(T))


def most_deferred(wide):
    """Most children that a walk of the tree can have deferred: on a path from the
    root, all internal children but the one descended to."""
    refs = wide[:, 24:28].copy().view(np.int32)
    inner = (refs >= 0) & (refs != EMPTY)
    most, stack = 0, [(0, 0)]
    while stack:
        node, held = stack.pop()
        kids = refs[node][inner[node]]
        held += max(0, len(kids) - 1)
        most = max(most, held)
        stack += [(int(k), held) for k in kids]
    return most


@pytest.mark.parametrize("kind,n_rays", [("slivers", 1), ("slivers", 65), ("slivers", 4099), ("nested", 1000),
                                         ("nested", 100_000), ("nested", 300_000)])
def test_deferred_children_outgrow_lds(kind, n_rays):
    import paper_2504_21719_amd as rt
    mesh = _scene(kind)
    scene = rt.scene_from_mesh(mesh)
    assert most_deferred(scene.export()["wide"]) >= STACK_LDS + 8
    pos = (0.3, -0.2, 3.0) if kind == "slivers" else (6.25, 6.25, 6.25)
    cfg = sg.Config(mesh, sg.Tx(pos, yaw=0.4, pattern=sg.PATTERN_DIRECTIONAL),
                    sg.Plane(1.5, -50.0, -50.0, 4.0, 4.0, 25, 25), sg.Params(3.5e9, n_rays, 2))
    ref = gpu_radio_map(cfg, scene_handle=scene, accel=rt.RT_ACCEL_BRUTE)
    for accel in (rt.RT_ACCEL_BVH4, rt.RT_ACCEL_BVH2):
        got = gpu_radio_map(cfg, scene_handle=scene, accel=accel)
        np.testing.assert_array_equal(got.hits, ref.hits)
        np.testing.assert_array_equal(got.cells, ref.cells)
        assert int(got.stats[4]) == 0
