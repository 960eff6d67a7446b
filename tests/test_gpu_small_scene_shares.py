"""The surface-area tree where a node's triangles are shared out over wavefronts:
sizes at the edges of 1 to 16 of them, nodes of very different sizes in one
level, and the one-block sort up to its largest size.  A tree does not depend
on who did what first."""
import numpy as np
import pytest

import scenegen as sg
from test_gpu_lbvh_structure import _mesh, check_scene

pytestmark = pytest.mark.gpu


def _grid(n):
    """Boxes' worth of equal triangles on a regular grid: centres that coincide
    on every axis."""
    i = np.arange(n)
    at = np.stack([i % 16, i // 16 % 16, i // 256], 1)[:, None, :] * 10.0
    t = np.array([[0.0, 0, 0], [6, 0, 1], [0, 6, 2]])
    return _mesh((at + t).reshape(-1, 3), np.arange(3 * n).reshape(n, 3))


def _lopsided(n, few):
    """`few` triangles far away from the others."""
    a = sg.random_soup(n - few, seed=n, extent=50.0, size=1.0)
    b = sg.random_soup(few, seed=few, extent=50.0, size=1.0)
    return _mesh(np.concatenate([a.vertices, b.vertices + np.float32(5000.0)]),
                 np.concatenate([a.triangles, b.triangles + len(a.vertices)]))


def _same_every_time(mesh):
    import paper_2504_21719_amd as rt
    dumps = []
    for _ in range(3):
        scene = rt.scene_from_mesh(mesh)      # named: its memory lives until the export
        dumps.append(scene.export())
    for d in dumps[1:]:
        for k in d:
            assert d[k].tobytes() == dumps[0][k].tobytes(), k


@pytest.mark.parametrize("n", [65, 128, 129, 192, 256, 257, 384, 511, 512, 513, 1024, 1026, 2047, 2050, 2352, 3890,
                               4096])
def test_sizes(n):
    for mesh in (sg.random_soup(n, seed=n), _grid(n)):
        check_scene(mesh)
        _same_every_time(mesh)


@pytest.mark.parametrize("n,few", [(4096, 2), (4096, 66), (3000, 300), (2200, 1030), (1300, 130)])
def test_nodes_of_different_sizes(n, few):
    mesh = _lopsided(n, few)
    check_scene(mesh)
    _same_every_time(mesh)
