"""Scenes whose trees are far deeper than a balanced one: Morton codes with a
single leading bit each (a chain), with many equal codes at its end.  The
builder queues a fixed number of levels of the 4-wide tree and goes on when
more are left; the traversal's spill area is sized from the depth."""
import numpy as np
import pytest

import scenegen as sg
from gpu_helpers import gpu_radio_map
from test_gpu_lbvh_structure import check_scene

pytestmark = pytest.mark.gpu


def _chain(bits, copies):
    """Small triangles at 2^i on every axis (one leading Morton bit each) and
    `copies` at the origin."""
    c = [np.eye(3)[a] * 2.0 ** i for i in range(bits) for a in range(3)] + [np.zeros(3)] * copies
    rng = np.random.default_rng(bits + copies)
    V = np.array(c)[:, None, :] + rng.uniform(-0.02, 0.02, (1, 3, 3))
    n = len(c)
    return sg.Scene(V.reshape(-1, 3).astype(np.float32), np.arange(3 * n, dtype=np.int32).reshape(n, 3),
                    np.zeros(n, np.int32), np.array([5.24]), np.array([0.12]), "chain")


@pytest.mark.parametrize("bits,copies", [(1, 0), (8, 1), (20, 1), (20, 33), (21, 3000)])
def test_chain(bits, copies):
    import paper_2504_21719_amd as rt
    mesh = _chain(bits, copies)
    info = check_scene(mesh)
    if bits >= 20:
        assert info.bvh_depth > 55
    cfg = sg.Config(mesh, sg.Tx((0.5, 0.4, 0.3)), sg.Plane(-1.0, -50.0, -50.0, 10.0, 10.0, 10, 10),
                    sg.Params(3.5e9, 3000, 2))
    ref = gpu_radio_map(cfg, accel=rt.RT_ACCEL_BRUTE)
    for accel in (rt.RT_ACCEL_BVH4, rt.RT_ACCEL_BVH2):
        got = gpu_radio_map(cfg, accel=accel)
        np.testing.assert_array_equal(got.hits, ref.hits)
        assert int(got.stats[4]) == 0


def test_invalid_meshes_are_refused():
    """Flags are read back once, after the whole build has run on stand-ins."""
    import torch
    import paper_2504_21719_amd as rt
    V = torch.tensor([[0, 0, 0], [1, 0, 0], [0, 1, 0], [1, 1, 1]], dtype=torch.float32, device="cuda")
    F = torch.tensor([[0, 1, 2], [1, 3, 2]] * 40, dtype=torch.int32, device="cuda")
    M = torch.zeros(80, dtype=torch.int32, device="cuda")
    rt.rt_build_scene(V, F, M, 1)
    for what, bad in (("vertex index", (V, F.index_fill(0, torch.tensor([17], device="cuda"), 4), M)),
                      ("vertex index", (V, F.index_fill(0, torch.tensor([0], device="cuda"), -1), M)),
                      ("material id", (V, F, M.index_fill(0, torch.tensor([79], device="cuda"), 1))),
                      ("non-finite", (V * float("nan"), F, M)), ("non-finite", (V / 0.0, F, M))):
        with pytest.raises(rt.RtError, match=what):
            rt.rt_build_scene(*bad, 1)
