"""Tapes in memory of the caller: argument checks (host), and the autograd
function's tapes from torch's allocator against tapes that own their memory."""
import ctypes as C

import numpy as np
import pytest

import scenegen as sg


def test_create_in_checks_its_memory_on_the_host():
    import paper_2504_21719_amd as rt
    L = rt.lib()
    p = rt.make_params(sg.Params(3.5e9, 100, 2))
    need = L.rt_tape_bytes(C.byref(p))
    buf = C.create_string_buffer(need + 64)
    base = (C.addressof(buf) + 15) & ~15            # never dereferenced by these calls
    h = C.c_void_p()
    for mem, n in ((base, need - 1), (base + 4, need), (0, need)):
        assert L.rt_tape_create_in(C.byref(p), C.c_void_p(mem), n, C.byref(h)) == rt.RT_EINVAL and not h.value
    assert L.rt_tape_create_in(C.byref(p), C.c_void_p(base), need, None) == rt.RT_EINVAL
    assert L.rt_tape_create_in(C.byref(p), C.c_void_p(base), need, C.byref(h)) == rt.RT_OK and h.value
    assert L.rt_tape_destroy(h) == rt.RT_OK
    empty = rt.make_params(sg.Params(3.5e9, 100, 2, ray_begin=5, ray_end=5))
    assert L.rt_tape_create_in(C.byref(empty), None, 0, C.byref(h)) == rt.RT_OK
    assert L.rt_tape_destroy(h) == rt.RT_OK


@pytest.mark.gpu
@pytest.mark.parametrize("n_rays,pol", [(1, sg.POL_V), (1000, sg.POL_DUAL), (200_003, sg.POL_V)])
@pytest.mark.parametrize("side_stream", [False, True])
def test_autograd_tapes_give_the_gradients_of_owned_tapes(n_rays, pol, side_stream):
    import torch
    import paper_2504_21719_amd as rt
    from paper_2504_21719_amd.autograd import radio_map
    cfg = sg.tiny_config(n_rays=n_rays, max_depth=3)
    cfg.tx = sg.Tx(cfg.tx.pos, yaw=0.2, pitch=-0.1, pattern=sg.PATTERN_DIRECTIONAL, pol=pol)
    scene = rt.scene_from_mesh(cfg.scene)
    npol = 2 if pol == sg.POL_DUAL else 1
    eps = torch.tensor(cfg.scene.eps_r, dtype=torch.float32, device="cuda", requires_grad=True)
    sig = torch.tensor(cfg.scene.sigma, dtype=torch.float32, device="cuda", requires_grad=True)
    ori = torch.tensor([0.2, -0.1, 0.0], dtype=torch.float64, requires_grad=True)
    up = torch.linspace(0.5, 2.0, npol * 10000, device="cuda").reshape(npol, 100, 100)
    torch.cuda.synchronize()
    got = []
    with torch.cuda.stream(torch.cuda.Stream() if side_stream else torch.cuda.current_stream()):
        for _ in range(3):      # the second and third tape reuse memory of the one before
            m = radio_map(eps, sig, ori, scene, cfg.tx, cfg.plane, cfg.params)
            got.append(torch.autograd.grad(m, (eps, sig, ori), up))
            del m
        torch.cuda.synchronize()
    tape = rt.rt_tape_create(cfg.params)
    out = torch.empty((npol, 100, 100), device="cuda")
    ge, gs, go = (torch.empty(n, device="cuda") for n in (1, 1, 3))
    args = (scene, eps.detach(), sig.detach(), cfg.tx, cfg.plane, cfg.params)
    rt.rt_radio_map(*args, out, tape=tape)
    rt.rt_radio_map_backward(*args, tape, up, ge, gs, go)
    for g in got:               # the adjoint sums in a fixed order
        assert torch.equal(g[0], ge) and torch.equal(g[1], gs)
        np.testing.assert_array_equal(g[2].numpy(), go.cpu().numpy().astype(np.float64))
