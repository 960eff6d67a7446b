"""Scenes of up to 4096 triangles take their 4-wide nodes from a tree split by
surface area: its structure at the edges of what a wavefront, the one-block
sort and the splitter hold, on degenerate input, and the hits through it."""
import numpy as np
import pytest

import scenegen as sg
from gpu_helpers import gpu_radio_map
from test_gpu_deep_tree import _chain
from test_gpu_lbvh_structure import _mesh, check_scene

pytestmark = pytest.mark.gpu


def _copies(n, seed=3):
    """n triangles at one place, of different sizes (no plane parts their centres)."""
    r = np.random.default_rng(seed).uniform(0.1, 5.0, (n, 1, 1))
    c = np.array([[-1.0, 0, 0], [1, 0, 0], [0, 1, 0]]) - np.array([0, 0.5, 0])
    return _mesh((r * c).reshape(-1, 3), np.arange(3 * n).reshape(n, 3))


def _line(n):
    """Centres at 1.02^i along a line: each split takes a few off the end."""
    rng = np.random.default_rng(n)
    c = 1.02 ** np.arange(n)[:, None, None] * np.array([1.0, 0.5, 0.25])
    return _mesh((c * (1 + 0.01 * rng.uniform(-1, 1, (n, 3, 3)))).reshape(-1, 3), np.arange(3 * n).reshape(n, 3))


@pytest.mark.parametrize("n", [2, 5, 63, 66, 128, 129, 2047, 2048, 2049, 4095, 4096, 4098])
def test_sizes(n):
    check_scene(sg.random_soup(n, seed=n))


@pytest.mark.parametrize("n", [2, 64, 65, 700, 4096])
def test_no_plane_parts_the_centres(n):
    check_scene(_copies(n))


@pytest.mark.parametrize("n", [60, 1000, 3500])
def test_one_sided(n):
    check_scene(_line(n))


def test_areas_beyond_fp32():
    rng = np.random.default_rng(7)
    V = rng.uniform(-1e38, 1e38, (3 * 300, 3)).astype(np.float32)
    check_scene(_mesh(V, np.arange(900).reshape(300, 3)))


def test_deep_tree_above_the_limit():
    check_scene(_chain(21, 5000))


def test_mixed_sizes_hits():
    """Triangles from a hundredth to all of the scene: the hits of both trees are
    those of brute force, and the 4-wide one is visited less than the other."""
    import paper_2504_21719_amd as rt
    a, b = sg.random_soup(1500, seed=1, extent=50.0, size=1.0), sg.random_soup(40, seed=2, extent=5.0, size=60.0)
    mesh = _mesh(np.concatenate([a.vertices, b.vertices]),
                 np.concatenate([a.triangles, b.triangles + len(a.vertices)]))
    cfg = sg.Config(mesh, sg.Tx((0.5, 0.4, 0.3)), sg.Plane(-1.0, -50.0, -50.0, 10.0, 10.0, 10, 10),
                    sg.Params(3.5e9, 20_000, 4))
    ref = gpu_radio_map(cfg, accel=rt.RT_ACCEL_BRUTE)
    visits = {}
    for accel in (rt.RT_ACCEL_BVH4, rt.RT_ACCEL_BVH2):
        got = gpu_radio_map(cfg, accel=accel)
        np.testing.assert_array_equal(got.hits, ref.hits)
        assert int(got.stats[4]) == 0
        visits[accel] = int(got.stats[2])
    assert visits[rt.RT_ACCEL_BVH4] < visits[rt.RT_ACCEL_BVH2]
