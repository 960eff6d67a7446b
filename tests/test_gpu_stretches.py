"""Calls whose deposits are not summed in the wavefronts (atomic strategy, or
lattice order) take their work from several stretches at once: every ray once,
and batched maps as single calls give them."""
import numpy as np
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu

LANES = 256 * 16 * 64        # lanes of the resident grid on 256 CUs
CONFIGS = [dict(order=2), dict(deposit=1), dict(order=2, deposit=1)]


@pytest.fixture(scope="module")
def site():
    import torch
    import paper_2504_21719_amd as rt
    cfg = sg.tiny_config()
    t = lambda a: torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda")
    return rt, torch, cfg, rt.scene_from_mesh(cfg.scene), t(cfg.scene.eps_r), t(cfg.scene.sigma)


@pytest.mark.parametrize("config", CONFIGS)
@pytest.mark.parametrize("lattice,first,last", [(4 * LANES - 64, 0, 4 * LANES - 64), (4 * LANES - 63, 0, 4 * LANES - 63),
                                                (9 * LANES + 333, 0, 9 * LANES + 333),
                                                (17 * LANES, 7 * LANES + 99, 17 * LANES - 5)])
def test_every_ray_once(site, config, lattice, first, last):
    rt, torch, cfg, scene, eps, sig = site
    rt.rt_set_launch_config(scene, **config)
    p = sg.Params(3.5e9, lattice, 1, ray_begin=first, ray_end=last)
    hits = torch.full((last - first, 2), -7, dtype=torch.int32, device="cuda")
    stats = torch.zeros(8, dtype=torch.int64, device="cuda")
    out = torch.empty((1, 100, 100), dtype=torch.float32, device="cuda")
    rt.rt_radio_map(scene, eps, sig, cfg.tx, cfg.plane, p, out, hits=hits, stats=stats)
    assert not bool((hits == -7).any()) and not bool((hits[:, 0] == -2).any()), "a ray was not traced"
    # a ray traced twice would count its segments twice
    assert int(stats[0]) == int((hits != -2).sum())


@pytest.mark.parametrize("config", CONFIGS)
@pytest.mark.parametrize("budgets", [[5 * LANES + 7], [3 * LANES + 1, 2 * LANES, 333], [LANES // 2 + 3] * 11])
def test_batched_maps_are_the_single_ones(site, config, budgets):
    rt, torch, cfg, scene, eps, sig = site
    txs = [sg.Tx((0.5 * i, -0.3 * i, 8.0 + 0.1 * i)) for i in range(len(budgets))]
    rt.rt_set_launch_config(scene, **config)
    out = torch.empty((len(txs), 1, 100, 100), dtype=torch.float32, device="cuda")
    rt.rt_radio_map_batched(scene, eps[None], sig[None], txs, budgets, cfg.plane, sg.Params(3.5e9, 1, 2), out)
    rt.rt_set_launch_config(scene)
    for i, (tx, n) in enumerate(zip(txs, budgets)):
        one = torch.empty((1, 100, 100), dtype=torch.float32, device="cuda")
        rt.rt_radio_map(scene, eps, sig, tx, cfg.plane, sg.Params(3.5e9, n, 2), one)
        a, b = out[i, 0].double().cpu().numpy(), one[0].double().cpu().numpy()
        # m crossings of similar size in a cell (up to some 5 n / 5000) added one
        # after another in two orders: m^(1/2) 2^-24 as the roundings fall, 2.2e-6
        # at m = 1300; a lost or doubled unit of 64 rays changes a cell by 64 / m
        np.testing.assert_allclose(a, b, rtol=2e-5, atol=2e-6 * float(b.max()))
