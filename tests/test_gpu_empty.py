"""Autograd with no query rows: empty outputs, and gradients that are empty or
zero, in the forward and the backward pass."""
import numpy as np
import pytest

from paper_2406_01713_amd import scenes as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("source", [False, True])
def test_autograd_without_queries(fp64, source):
    import torch
    from paper_2406_01713_amd.autograd import wos_u
    dt = torch.float64 if fp64 else torch.float32
    s = S.scene_spheres(3, m_sph=20, n_queries=1, sigma=0.0 if source else 1.0)
    if source:  # no sigma derivative at sigma = 0: the pass without the derivatives
        s = S.with_source(s, np.zeros(3))
    x = torch.empty(0, 3, dtype=dt, device="cuda", requires_grad=True)
    sg = torch.tensor(s["sigma"], dtype=dt, requires_grad=True)
    gg = torch.tensor(1.0, dtype=dt, requires_grad=True)
    u, g = wos_u(x, sg, gg, s, 64, 1e-3, 1)
    assert u.shape == (0,) and g.shape == (0, 3)
    if not source:
        u.sum().backward()
        assert x.grad.shape == (0, 3) and sg.grad.item() == 0.0 and gg.grad.item() == 0.0
