"""|alpha|^2 of a transmit array, ray by ray, against FP64: odd and even element
counts, offsets from zero to many wavelengths, every quadrant, single and
batched."""
import numpy as np
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu

FREQ = 3.5e9
LAM = 299792458.0 / FREQ


def _directions(N):
    n = np.arange(N, dtype=np.uint64)
    turns = ((n * np.uint64(0x9e3779b97f4a7c16)) >> np.uint64(11)).astype(np.float64) * 2.0 ** -53
    # the lattice rounds the sum once; near the poles it tells
    z = (1 - np.arange(N).astype(np.longdouble) * np.longdouble(2.0 / (N - 1))).astype(np.float64)
    s = np.sqrt((1.0 - z) * (1.0 + z))
    return np.stack([s * np.cos(2 * np.pi * turns), s * np.sin(2 * np.pi * turns), z], 1)


@pytest.mark.parametrize("n,extent", [(1, 0.0), (1, 0.3), (2, 1.0), (3, 40.0), (64, 8.0), (65, 1e4)])
def test_gain_of_every_ray(n, extent):
    import torch
    import paper_2504_21719_amd as rt
    cfg = sg.tiny_config()
    N = 20_000
    rng = np.random.default_rng(n)
    pos = rng.uniform(-extent, extent, (n, 3)) * LAM
    u = (np.exp(2j * np.pi * rng.uniform(size=n)) / np.sqrt(n)).astype(np.complex64)
    scene = rt.scene_from_mesh(cfg.scene)
    t = lambda a: torch.tensor(np.asarray(a), dtype=torch.float32, device="cuda")
    eps, sig = t(cfg.scene.eps_r), t(cfg.scene.sigma)
    w = []
    for array in (None, sg.TxArray(pos, u)):
        wt = torch.zeros((N, 1), dtype=torch.float32, device="cuda")
        out = torch.empty((1, 100, 100), dtype=torch.float32, device="cuda")
        rt.rt_radio_map(scene, eps, sig, sg.Tx(cfg.tx.pos, array=array), cfg.plane, sg.Params(FREQ, N, 0), out, weights=wt)
        w.append(wt[:, 0].double().cpu().numpy())
    one = out
    alpha = np.exp(2j * np.pi / LAM * (_directions(N) @ pos.T)) @ u.astype(np.complex128)
    # FP32 sums of n terms of size n^-1/2, each with 2.5e-7 of sine, cosine,
    # product and sum: |alpha| <= n^1/2 to n^1/2 2.5e-7 n^1/2, its square to 5e-7 n^3/2
    # at the very worst, n at random; 2e-7 for the weight itself
    tol = (1e-6 * n + 2e-7 * np.abs(alpha) ** 2) * w[0]
    assert (w[0] > 0).sum() > 1000
    assert np.all(np.abs(w[1] - w[0] * np.abs(alpha) ** 2) <= tol)
    two = torch.empty((2, 1, 100, 100), dtype=torch.float32, device="cuda")
    rt.rt_radio_map_batched(scene, eps[None], sig[None], [sg.Tx(cfg.tx.pos, array=array), sg.Tx(cfg.tx.pos)], [N, N],
                            cfg.plane, sg.Params(FREQ, 1, 0), two)
    a, b = two[0].double().cpu().numpy(), one.double().cpu().numpy()
    np.testing.assert_allclose(a, b, rtol=2e-5, atol=2e-6 * float(b.max()))
