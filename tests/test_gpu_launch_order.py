"""The coherent launch order is a permutation of the rays to trace, for whole
chunks, every kind of rest and sub-ranges, single and batched."""
import numpy as np
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu

# around the smallest ordered count, the chunk sizes (610, 987, 1597, ...) and
# their sums, and rests of every length down to one ray
COUNTS = [1, 511, 512, 513, 609, 610, 611, 753, 754, 755, 986, 987, 1597 * 3, 1597 * 3 + 144, 1597 * 3 + 143,
          2584 * 7 + 987 + 377 + 144 + 5, 100_003]


@pytest.mark.parametrize("count", COUNTS)
@pytest.mark.parametrize("begin", [0, 37])
def test_every_ray_once(count, begin):
    import torch
    import paper_2504_21719_amd as rt
    cfg = sg.tiny_config()
    scene = rt.scene_from_mesh(cfg.scene)
    eps = torch.tensor(cfg.scene.eps_r, dtype=torch.float32, device="cuda")
    sig = torch.tensor(cfg.scene.sigma, dtype=torch.float32, device="cuda")
    p = sg.Params(3.5e9, count + begin, 1, ray_begin=begin)
    hits = torch.full((count, 2), -7, dtype=torch.int32, device="cuda")
    w = torch.full((count, 2), -7.0, dtype=torch.float32, device="cuda")
    stats = torch.zeros(8, dtype=torch.int64, device="cuda")
    out = torch.empty((1, 100, 100), dtype=torch.float32, device="cuda")
    rt.rt_radio_map(scene, eps, sig, cfg.tx, cfg.plane, p, out, hits=hits, weights=w, stats=stats)
    h = hits.cpu().numpy()
    assert not np.any(h == -7) and not np.any(h[:, 0] == -2), "a ray was not traced"
    # a ray traced twice would count its segments twice
    assert int(stats[0]) == int(np.sum(h != -2))
    rt.rt_set_launch_config(scene, order=2)
    hits2, w2 = torch.full_like(hits, -7), torch.full_like(w, -7.0)
    rt.rt_radio_map(scene, eps, sig, cfg.tx, cfg.plane, p, out, hits=hits2, weights=w2)
    assert torch.equal(hits, hits2) and torch.equal(w, w2)      # the same ray at every index


def test_batched_maps_in_both_orders():
    """Budgets of every kind of rest in one call: each map as in lattice order."""
    import torch
    import paper_2504_21719_amd as rt
    cfg = sg.tiny_config()
    scene = rt.scene_from_mesh(cfg.scene)
    txs = [sg.Tx((0.5 * i, -0.3 * i, 8.0 + 0.1 * i)) for i in range(len(COUNTS))]
    dev = dict(dtype=torch.float32, device="cuda")
    eps, sig = torch.tensor([[5.24], [4.0]], **dev), torch.tensor([[0.12], [0.2]], **dev)
    got = []
    for order in (1, 2):
        rt.rt_set_launch_config(scene, order=order)
        for e, s in ((eps[:1], sig[:1]), (eps, sig)):            # the map kernel, the geometry tape
            out = torch.empty((len(txs), e.shape[0], 100, 100), **dev)
            rt.rt_radio_map_batched(scene, e.contiguous(), s.contiguous(), txs, COUNTS, cfg.plane,
                                    sg.Params(3.5e9, 1, 2), out)
            got.append(out.cpu().numpy())
    for a, b in ((got[0], got[2]), (got[1], got[3])):
        # the same crossings summed in another order: 2e-5 covers a few hundred in a cell
        np.testing.assert_allclose(a, b, rtol=2e-5, atol=1e-7 * float(b.max()))
