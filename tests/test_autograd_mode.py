"""Which call of the library the autograd function's forward pass makes: the
estimate alone where no gradient can be asked for (grad mode off, or inputs that
require none), the estimate with its derivatives otherwise.  The library's calls
are replaced, so no GPU is needed."""
import contextlib

import pytest


@pytest.mark.parametrize("mode,requires,want", [
    ("grad", (True, False, False), "jac"), ("grad", (False, True, False), "jac"), ("grad", (False, False, True), "jac"),
    ("grad", (False, False, False), "estimate"), ("no_grad", (True, True, True), "estimate"),
    ("inference", (True, True, True), "estimate"), ("no_grad", (False, False, False), "estimate")])
def test_forward_call(monkeypatch, mode, requires, want):
    import torch
    from paper_2406_01713_amd import autograd as A
    from paper_2406_01713_amd import scenes as S
    calls = []

    class Dom:
        has_source = False

        def __init__(self, scene):
            pass

    monkeypatch.setattr(A.B, "Domain", Dom)
    monkeypatch.setattr(A.B, "wos_estimate", lambda dom, x, n, s, e, seed, u, g, *a, **k: calls.append("estimate"))
    monkeypatch.setattr(A.B, "wos_estimate_jac", lambda dom, x, n, s, e, seed, u, g, *a, **k: calls.append("jac"))
    monkeypatch.setattr(A.WoSFunction, "_cache", {})
    s = S.scene_spheres(3, m_sph=4, n_queries=2)
    x = torch.tensor(s["queries"], requires_grad=requires[0])
    sg, gg = (torch.tensor(1.0, dtype=torch.float64, requires_grad=r) for r in requires[1:])
    with {"grad": contextlib.nullcontext, "no_grad": torch.no_grad, "inference": torch.inference_mode}[mode]():
        for fn in (A.wos_u, A.WoSFunction.apply):
            u, g = fn(x, sg, gg, s, 8, 1e-3, 1)
            assert u.requires_grad == (want == "jac") and not g.requires_grad
    assert calls == [want, want]
