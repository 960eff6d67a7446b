"""t_min = -0.0 is accepted and means 0: a box that holds a ray's origin is then
entered at t_min, and a zero's sign must not change its place among the boxes
to visit."""
import numpy as np
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu


def _triangle(x, size):
    return np.array([[x, -size, -size], [x, size, -size], [x, 0.0, 1.5 * size]])


def _scene():
    """Along +x: a pair around the origin, one triangle much larger than the
    others, and two more pairs beyond it."""
    T = np.array([_triangle(x, s) for x, s in ((0.6, 0.5), (-0.6, 0.5), (5.0, 50.0), (10.0, 6.0), (12.0, 6.0),
                                               (30.0, 6.0), (33.0, 6.0))])
    n = len(T)
    return sg.Scene(T.reshape(-1, 3).astype(np.float32), np.arange(3 * n, dtype=np.int32).reshape(n, 3),
                    np.zeros(n, np.int32), np.array([5.24]), np.array([0.12]), "pairs")


@pytest.mark.parametrize("n_rays", [64, 500, 20_000])
def test_negative_zero_is_zero(n_rays):
    import torch
    import paper_2504_21719_amd as rt
    mesh = _scene()
    scene = rt.scene_from_mesh(mesh)
    # the case at hand: a leaf and internal children in the root, so that a hit
    # in the leaf can lie nearer than one child and farther than another
    root = scene.export()["wide"][0, 24:28].copy().view(np.int32)
    assert (root < 0).sum() == 1 and ((root >= 0) & (root < 0x7fffffff)).sum() == 3
    t = lambda a: torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda")
    eps, sig = t(mesh.eps_r), t(mesh.sigma)
    tx, plane = sg.Tx((0.0, 0.0, 0.0)), sg.Plane(-0.1, -5.0, -5.0, 1.0, 1.0, 10, 10)
    hits, maps = {}, {}
    for accel in (rt.RT_ACCEL_BRUTE, rt.RT_ACCEL_BVH2, rt.RT_ACCEL_BVH4):
        for sign in (1.0, -1.0):
            p = sg.Params(3.5e9, n_rays, 0, t_min=sign * 0.0)
            h = torch.empty((n_rays, 1), dtype=torch.int32, device="cuda")
            out = torch.empty((1, 10, 10), dtype=torch.float32, device="cuda")
            rt.rt_radio_map(scene, eps, sig, tx, plane, p, out, hits=h, accel=accel)
            hits[accel, sign], maps[accel, sign] = h.cpu().numpy(), out.cpu().numpy()
    ref = hits[rt.RT_ACCEL_BRUTE, 1.0]
    assert (ref == 0).any()
    for key, h in hits.items():
        np.testing.assert_array_equal(h, ref, err_msg=str(key))
    for sign in (1.0, -1.0):
        out = torch.empty((2, 1, 10, 10), dtype=torch.float32, device="cuda")
        rt.rt_radio_map_batched(scene, eps[None], sig[None], [tx, tx], [n_rays, n_rays], plane,
                                sg.Params(3.5e9, 1, 0, t_min=sign * 0.0), out)
        # the same crossings (some hundreds in a cell) summed in another order
        np.testing.assert_allclose(out[0].cpu().numpy(), maps[rt.RT_ACCEL_BRUTE, 1.0], rtol=2e-5,
                                   atol=1e-6 * float(out.max()))
