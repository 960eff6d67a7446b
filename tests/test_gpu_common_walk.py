"""The 4-wide traversal that a wavefront's lanes walk together, and its hand-over
to the per-lane loop, against testing every triangle (same triangle test, so
hits are equal; maps differ by FP32 summation order only)."""
import numpy as np
import pytest

import scenegen as sg
from gpu_helpers import gpu_radio_map

pytestmark = pytest.mark.gpu


def _scene(kind):
    if kind == "quad":          # every wavefront stays together
        return sg.ground_quad(50.0)
    if kind == "soup":          # neighbouring rays part at every bounce
        return sg.random_soup(700, seed=3, extent=20.0, size=4.0)
    # triangles through the whole volume: nearly every child box is entered,
    # so that the deferred children outgrow the 16 stack entries held in LDS
    return sg.random_soup(600, seed=4, extent=2.0, size=60.0)


@pytest.mark.parametrize("kind", ["quad", "soup", "overlap"])
@pytest.mark.parametrize("n_rays", [1, 63, 64, 65, 4099])
@pytest.mark.parametrize("pol", [sg.POL_V, sg.POL_DUAL])
def test_common_walk_matches_every_triangle(kind, n_rays, pol):
    import paper_2504_21719_amd as rt
    cfg = sg.Config(_scene(kind), sg.Tx((0.3, -0.2, 9.0), yaw=0.4, pattern=sg.PATTERN_DIRECTIONAL, pol=pol),
                    sg.Plane(1.5, -50.0, -50.0, 4.0, 4.0, 25, 25), sg.Params(3.5e9, n_rays, 3))
    ref = gpu_radio_map(cfg, accel=rt.RT_ACCEL_BRUTE, records=True)
    got = gpu_radio_map(cfg, accel=rt.RT_ACCEL_BVH4, records=True)
    np.testing.assert_array_equal(got.hits, ref.hits)
    np.testing.assert_array_equal(got.cells, ref.cells)
    assert int(got.stats[4]) == 0
    # the same call without records (fields instead of transfer matrices);
    # 2e-5: up to a few hundred crossings per cell summed in another order,
    # and fields formed in another order over four reflections
    plain = gpu_radio_map(cfg, accel=rt.RT_ACCEL_BVH4, records=False)
    np.testing.assert_allclose(plain.map, ref.map, rtol=2e-5, atol=1e-6 * max(float(ref.map.max()), 1e-30))
