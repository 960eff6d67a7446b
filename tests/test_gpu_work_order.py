"""The work queues hand out every ray exactly once: at the widths and grids of
small calls, with several units per wavefront, for parts of a lattice on
either side of its equator, and for several transmitters."""
import numpy as np
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu

LANES = 256 * 16 * 64        # lanes of the resident grid on 256 CUs

# (rays of the lattice, first, last): around the narrowest wavefronts, the
# widths, the last count at which every wavefront has one unit, whole and
# ragged numbers of units, units of two and of four wavefronts
RANGES = [(n, 0, n) for n in (1, 7, 8, 9, 65, LANES // 8 - 57, LANES // 8 - 56, LANES // 8 - 55, LANES // 2,
                              LANES - 449, LANES - 448, LANES - 447, LANES + 1, 4 * LANES + 1000, 33 * LANES + 17,
                              65 * LANES - 63)]
# the equator outside the part, at its ends, and off its middle
RANGES += [(4 * LANES, 0, 2 * LANES - 5), (4 * LANES, 2 * LANES, 4 * LANES), (4 * LANES, 2 * LANES - 64, 4 * LANES - 3),
           (4 * LANES, 2 * LANES + 999, 4 * LANES), (4 * LANES, LANES // 3, 2 * LANES + 70)]


def _scene():
    import torch
    import paper_2504_21719_amd as rt
    cfg = sg.tiny_config()
    t = lambda a: torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda")
    return rt, torch, cfg, rt.scene_from_mesh(cfg.scene), t(cfg.scene.eps_r), t(cfg.scene.sigma)


def _traced_once(lattice, first, last):
    rt, torch, cfg, scene, eps, sig = _scene()
    p = sg.Params(3.5e9, lattice, 1, ray_begin=first, ray_end=last)
    hits = torch.full((last - first, 2), -7, dtype=torch.int32, device="cuda")
    stats = torch.zeros(8, dtype=torch.int64, device="cuda")
    out = torch.empty((1, 100, 100), dtype=torch.float32, device="cuda")
    rt.rt_radio_map(scene, eps, sig, cfg.tx, cfg.plane, p, out, hits=hits, stats=stats)
    assert not bool((hits == -7).any()) and not bool((hits[:, 0] == -2).any()), "a ray was not traced"
    # a ray traced twice would count its segments twice
    assert int(stats[0]) == int((hits != -2).sum())


@pytest.mark.parametrize("lattice,first,last", RANGES)
def test_every_ray_once(lattice, first, last):
    _traced_once(lattice, first, last)


@pytest.mark.parametrize("queues", ["1", "7", "32", "256"])
@pytest.mark.parametrize("claim", ["64", "192", "4096"])
def test_every_ray_once_with_overrides(monkeypatch, queues, claim):
    monkeypatch.setenv("RTMAP_QUEUES", queues)
    monkeypatch.setenv("RTMAP_CLAIM", claim)
    _traced_once(5 * LANES + 333, 0, 5 * LANES + 333)


@pytest.mark.parametrize("budgets", [[3], [LANES + 5], [700, 65, 1], [2 * LANES + 1, LANES, 333],
                                     [34 * LANES + 11, LANES + 3, 999]])
def test_batched_maps_are_the_single_ones(budgets):
    rt, torch, cfg, scene, eps, sig = _scene()
    txs = [sg.Tx((0.5 * i, -0.3 * i, 8.0 + 0.1 * i)) for i in range(len(budgets))]
    out = torch.empty((len(txs), 1, 100, 100), dtype=torch.float32, device="cuda")
    rt.rt_radio_map_batched(scene, eps[None], sig[None], txs, budgets, cfg.plane, sg.Params(3.5e9, 1, 2), out)
    for i, (tx, n) in enumerate(zip(txs, budgets)):
        one = torch.empty((1, 100, 100), dtype=torch.float32, device="cuda")
        rt.rt_radio_map(scene, eps, sig, tx, cfg.plane, sg.Params(3.5e9, n, 2), one)
        a, b = out[i, 0].double().cpu().numpy(), one[0].double().cpu().numpy()
        # m equal-sized crossings added one after another in two orders, each
        # rounding to 2^-24: m 2^-24 apart at worst, m up to 34 LANES / 5000 in
        # a cell before, m^(1/2) 2^-24 (2.6e-6) as they fall; a lost or doubled
        # unit of 64 rays changes a whole cell
        np.testing.assert_allclose(a, b, rtol=2e-5, atol=2e-6 * float(b.max()))


@pytest.mark.parametrize("lattice,first,last", [(LANES // 4, 0, LANES // 4), (LANES // 4 + 513, 0, LANES // 4 + 513),
                                                (LANES // 4 + 700, 0, LANES // 4 + 700),
                                                (LANES // 2 + 9, 0, LANES // 2 + 9), (LANES, 300, LANES - 5),
                                                (LANES, LANES // 2 - 100, LANES - 5), (LANES, 0, LANES // 2 + 100),
                                                (LANES - 447, 0, LANES - 447), (LANES + 1, 0, LANES + 1),
                                                (3 * LANES + 77, 0, 3 * LANES + 77), (6 * LANES, 0, 6 * LANES),
                                                (6 * LANES + 1, 0, 6 * LANES + 1), (4 * LANES, LANES + 99, 4 * LANES),
                                                (4 * LANES, 2 * LANES - 32768, 4 * LANES - 5),
                                                (4 * LANES, 2 * LANES - 32700, 4 * LANES - 5),
                                                (4 * LANES, 0, 2 * LANES + 32768 + 64)])
def test_every_ray_once_on_a_large_tree(large_scene, lattice, first, last):
    """First units of 16 rays at the equator, up to six units per wavefront and
    with room on both sides of it."""
    rt, torch, cfg, scene, eps, sig = large_scene
    p = sg.Params(3.5e9, lattice, 0, ray_begin=first, ray_end=last)
    hits = torch.full((last - first, 1), -7, dtype=torch.int32, device="cuda")
    stats = torch.zeros(8, dtype=torch.int64, device="cuda")
    out = torch.empty((1, cfg.plane.H, cfg.plane.W), dtype=torch.float32, device="cuda")
    rt.rt_radio_map(scene, eps, sig, cfg.tx, cfg.plane, p, out, hits=hits, stats=stats)
    assert not bool((hits == -7).any()) and not bool((hits == -2).any()), "a ray was not traced"
    assert int(stats[0]) == last - first


@pytest.fixture(scope="module")
def large_scene():
    import torch
    import paper_2504_21719_amd as rt
    cfg = sg.large_config(1000)
    t = lambda a: torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda")
    return rt, torch, cfg, rt.scene_from_mesh(cfg.scene), t(cfg.scene.eps_r), t(cfg.scene.sigma)
