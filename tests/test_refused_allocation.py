"""Device memory that the driver refuses: torch's allocator, which keeps the
autograd function's tapes, gives back what it does not use and the call is made
again; a refusal is reported once, by the call that it befell."""
import types

import pytest

import scenegen as sg


class _Library:
    """Entry points that refuse the first `times` calls."""

    def __init__(self, status, times):
        self.status, self.times, self.calls = status, times, 0

    def __getattr__(self, name):
        def entry(*args):
            self.calls += 1
            return self.status if self.calls <= self.times else 0
        return {"rt_last_error": lambda: b"refused", "rt_tape_bytes": lambda p: 64}.get(name, entry)


@pytest.mark.parametrize("name", ["build", "tape", "batched", "backward"])
@pytest.mark.parametrize("status,times,calls", [("RT_ENOMEM", 1, 2), ("RT_ENOMEM", 9, 2), ("RT_EDEVICE", 1, 1),
                                                ("RT_OK", 0, 1)])
def test_refused_memory_is_asked_for_again(monkeypatch, name, status, times, calls):
    import torch
    import paper_2504_21719_amd as rt
    L = _Library(getattr(rt, status), times)
    given_back = []
    monkeypatch.setattr(rt, "lib", lambda: L)
    monkeypatch.setattr(rt, "_ptrs", lambda *specs: [None] * len(specs))
    monkeypatch.setattr(rt, "_stream", lambda stream=None: None)
    monkeypatch.setattr(torch.cuda, "empty_cache", lambda: given_back.append(L.calls))
    t = torch.zeros(3, 3)
    scene = types.SimpleNamespace(handle=1, n_materials=1)
    plane, p, tx = sg.Plane(0.0, 0.0, 0.0, 1.0, 1.0, 3, 3), sg.Params(3.5e9, 10, 1), sg.Tx((0.0, 0.0, 1.0))
    call = {
        "build": lambda: rt.rt_build_scene(t, t.int(), t[0].int(), 1),
        "tape": lambda: rt.rt_tape_create(p),
        "batched": lambda: rt.rt_radio_map_batched(scene, t[:1, :1], t[:1, :1], [tx], [10], plane, p, t),
        "backward": lambda: rt.rt_radio_map_backward(scene, t[0, :1], t[0, :1], tx, plane, p,
                                                     types.SimpleNamespace(handle=1), t),
    }[name]
    if times >= calls:
        with pytest.raises(rt.RtError) as e:
            call()
        assert e.value.status == getattr(rt, status)
    else:
        call()
    assert L.calls == calls and given_back == ([1] if calls == 2 else [])


@pytest.mark.gpu
def test_a_refusal_is_reported_once():
    import torch
    import paper_2504_21719_amd as rt
    cfg = sg.tiny_config(n_rays=1000, max_depth=1)
    scene = rt.scene_from_mesh(cfg.scene)
    eps = torch.tensor(cfg.scene.eps_r, dtype=torch.float32, device="cuda")
    sig = torch.tensor(cfg.scene.sigma, dtype=torch.float32, device="cuda")
    out = torch.empty((1, cfg.plane.H, cfg.plane.W), dtype=torch.float32, device="cuda")
    with pytest.raises(rt.RtError) as e:
        rt.rt_tape_create(sg.Params(3.5e9, 1 << 40, 8))          # 630 TB
    assert e.value.status == rt.RT_ENOMEM
    rt.rt_radio_map(scene, eps, sig, cfg.tx, cfg.plane, cfg.params, out)
    assert float(out.sum()) > 0
