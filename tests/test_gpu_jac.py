"""wos_estimate_jac: one pass gives wos_estimate's outputs and the derivatives
wos_backward weights, and the autograd function built on it gives
wos_backward's products."""
import numpy as np
import pytest

from paper_2406_01713_amd import scenes as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch  # noqa: F401  (the HIP runtime the library binds to)
    from paper_2406_01713_amd import binding
    return binding


@pytest.mark.parametrize("d", [2, 7])
@pytest.mark.parametrize("fp64", [False, True])
def test_jac_matches_estimate_and_backward(B, d, fp64):
    import torch
    from paper_2406_01713_amd.autograd import wos_u
    dt = torch.float64 if fp64 else torch.float32
    s = S.scene_spheres(d, m_sph=40, n_queries=5, n_walks=257, sigma=2.0, eps=1e-3)
    s = S.with_bdata(s, 2, ak=S.plane_wave_k(d, 2.0))
    x = torch.tensor(s["queries"], dtype=dt, device="cuda")
    Q, n, seed = len(x), 257, 12
    e = lambda *sh: torch.empty(*sh, dtype=dt, device="cuda")  # noqa: E731
    f = lambda *sh: torch.empty(*sh, dtype=torch.float64, device="cuda")  # noqa: E731
    opt = B.options(fp64)
    dom = B.Domain(s)
    u, g, st, u2, g2, st2, jac = e(Q), e(Q, d), f(Q, d + 4), e(Q), e(Q, d), f(Q, d + 4), f(Q, d + 2)
    B.wos_estimate(dom, x, n, 2.0, 1e-3, seed, u, g, st, opt=opt)
    B.wos_estimate_jac(dom, x, n, 2.0, 1e-3, seed, u2, g2, st2, jac, opt=opt)
    assert torch.equal(u, u2) and torch.equal(g, g2) and torch.equal(st, st2)
    ub = torch.tensor(np.random.default_rng(1).normal(size=Q), dtype=dt, device="cuda")
    dx, ds, dg, dq = e(Q, d), f(1), f(1), f(Q, 2)
    B.wos_backward(dom, x, n, 2.0, 1e-3, seed, ub, dx, ds, dg, dq, opt=opt)
    assert torch.equal(dq, jac[:, d:])
    assert torch.equal(dx, (ub.double()[:, None] * jac[:, :d]).to(dt))
    xa = x.clone().requires_grad_(True)
    sg, gg = torch.tensor(2.0, dtype=dt, requires_grad=True), torch.tensor(0.0, dtype=dt, requires_grad=True)
    ua, ga = wos_u(xa, sg, gg, s, n, 1e-3, seed)
    ua.backward(ub)
    assert torch.equal(ua.detach(), u) and torch.equal(ga, g) and torch.equal(xa.grad, dx)
    # sums of 5 products in another order: FP64 rounding, then the type's
    tol = 1e-13 if fp64 else 1e-6
    for got, want in ((sg.grad, ds), (gg.grad, dg)):
        assert abs(got.item() - want.item()) <= tol * (ub.abs().double()[:, None] * jac[:, d:].abs()).sum().item()


def test_jac_rejects_what_backward_rejects(B):
    import torch
    s = S.scene_ball_source(2, sigma=0.0, queries=np.array([[0.3, 0.1]]))
    dom = B.Domain(s)
    x = torch.tensor(s["queries"], dtype=torch.float32, device="cuda")
    u, g, jac = torch.empty(1, device="cuda"), torch.empty(1, 2, device="cuda"), torch.empty(1, 4, dtype=torch.float64, device="cuda")
    with pytest.raises(B.WosError):
        B.wos_estimate_jac(dom, x, 8, 0.0, 1e-3, 1, u, g, None, jac)  # no sigma derivative at sigma = 0
    with pytest.raises(B.WosError):
        B.wos_estimate_jac(dom, x, 8, 1.0, 1e-3, 1, u, g, None, None)
