"""Batched calls on a tree larger than an L2 against single ones: several
transmitters that go through stretches of their lattices at once, and one whose
first units are of 16 rays."""
import numpy as np
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu

LANES = 256 * 16 * 64        # lanes of the resident grid on 256 CUs


@pytest.fixture(scope="module")
def terrain():
    import torch
    import paper_2504_21719_amd as rt
    cfg = sg.large_config(1000)
    t = lambda a: torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda")
    return rt, torch, cfg, rt.scene_from_mesh(cfg.scene), t(cfg.scene.eps_r), t(cfg.scene.sigma)


def _compare(terrain, budgets, samples, depth=2):
    rt, torch, cfg, scene, eps, sig = terrain
    x, y, z = cfg.tx.pos
    txs = [sg.Tx((x + 3.0 * i, y - 2.0 * i, z + 5.0 + 0.1 * i)) for i in range(len(budgets))]
    H, W = cfg.plane.H, cfg.plane.W
    out = torch.empty((len(txs), samples, H, W), dtype=torch.float32, device="cuda")
    rep = lambda v: v[None].repeat(samples, 1).contiguous()
    rt.rt_radio_map_batched(scene, rep(eps), rep(sig), txs, budgets, cfg.plane, sg.Params(3.5e9, 1, depth), out)
    for i, (tx, n) in enumerate(zip(txs, budgets)):
        one = torch.empty((1, H, W), dtype=torch.float32, device="cuda")
        rt.rt_radio_map(scene, eps, sig, tx, cfg.plane, sg.Params(3.5e9, n, depth), one)
        b = one[0].double().cpu().numpy()
        assert (b > 0).sum() > min(1000, n // 2)
        for s in range(samples):
            # the same crossings summed in another order, the samples' fields also
            # formed in another order over two reflections: 2e-5 and, for cells of
            # many crossings, 2e-6 of the largest; a lost or doubled unit of rays
            # changes a cell by its share of them
            np.testing.assert_allclose(out[i, s].double().cpu().numpy(), b, rtol=2e-5, atol=2e-6 * float(b.max()))


@pytest.mark.parametrize("samples", [1, 2])
@pytest.mark.parametrize("budgets", [[50_000] * 24, [2 * LANES + 5, 2 * LANES, LANES + 7], [LANES // 3] * 13 + [999],
                                     [LANES // 3] * 5, [LANES // 2 + 1] * 3])
def test_several_transmitters(terrain, budgets, samples):
    _compare(terrain, budgets, samples)


@pytest.mark.parametrize("samples", [1, 2])
@pytest.mark.parametrize("n", [LANES // 2 + 9, 2 * LANES + 1, 5 * LANES - 77])
def test_one_transmitter(terrain, n, samples):
    _compare(terrain, [n], samples)


@pytest.mark.parametrize("refill", [8, 48, 64])
def test_first_units_and_refills(terrain, refill):
    """Whatever the refill threshold, the narrow first units hand out every ray."""
    rt, torch, cfg, scene, eps, sig = terrain
    n = 2 * LANES + 333
    rt.rt_set_launch_config(scene, refill=refill)
    hits = torch.full((n, 1), -7, dtype=torch.int32, device="cuda")
    stats = torch.zeros(8, dtype=torch.int64, device="cuda")
    out = torch.empty((1, cfg.plane.H, cfg.plane.W), dtype=torch.float32, device="cuda")
    rt.rt_radio_map(scene, eps, sig, cfg.tx, cfg.plane, sg.Params(3.5e9, n, 0), out, hits=hits, stats=stats)
    rt.rt_set_launch_config(scene)
    assert not bool((hits == -7).any()) and not bool((hits == -2).any()) and int(stats[0]) == n
