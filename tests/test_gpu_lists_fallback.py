"""Walks of environments whose cell lists do not fit: one cell would list more
obstacles than its header can count, so the steps scan clusters.  A bundle of
equal obstacles outside the region that matters brings any scene there; the
cluster scan's variants (pairs with and without the bounding-box test, a queue
that overflows, whole-wave and vector-ALU scans) then give the full scan's
walks, for spheres and boxes, in few and many dimensions."""
import numpy as np
import pytest

from paper_2406_01713_amd import scenes as S

pytestmark = pytest.mark.gpu

# more equal obstacles than the 2160 entries a cell's count byte can say
BUNDLE = 2200


@pytest.fixture(scope="module")
def B():
    import torch  # noqa: F401  (the HIP runtime the library binds to)
    from paper_2406_01713_amd import binding
    return binding


def _scene(d, boxes, m, dense):
    """Obstacles in [-3, 3]^d (dense: half of them packed around the origin, so
    that every walker of a wave needs every cluster there) and the bundle at a
    corner."""
    rng = np.random.default_rng(100 * d + 10 * boxes + m)
    c = rng.uniform(-2.5, 2.5, size=(m, d))
    r = rng.uniform(0.05, 0.3, size=m)
    if dense:
        c[: m // 2] = rng.uniform(-0.5, 0.5, size=(m // 2, d))
        r[: m // 2] = rng.uniform(0.01, 0.02, size=m // 2)
    c = np.concatenate([c, np.full((BUNDLE, d), 2.9)])
    r = np.concatenate([r, np.full(BUNDLE, 0.02)])
    s = S._empty(d)
    if boxes:
        s.update(box_c=c, box_h=np.repeat(r[:, None], d, axis=1))
    else:
        s.update(sph_c=c, sph_r=r)
    s.update(d=d, goal_c=np.full(d, -2.0), goal_r=0.4, outer=S.box_outer(d, 3.0),
             bdata=S._bdata(0, d, g_goal=1.0, g_obs=0.5, g_outer=0.25), sigma=1.0, eps=1e-3, n_walks=128, seed=5)
    s["queries"] = np.concatenate([rng.uniform(-0.4, 0.4, size=(3, d)), rng.uniform(-2.0, 2.0, size=(3, d)),
                                   [np.full(d, 2.8)]])
    return s


CASES = [(2, False, 200, False), (3, False, 1536, True), (3, True, 1536, True), (5, True, 300, False),
         (6, False, 300, False), (7, True, 200, False), (8, False, 400, False)]


@pytest.mark.parametrize("d,boxes,m,dense", CASES)
def test_cluster_scan_gives_the_full_scans_walks(B, d, boxes, m, dense):
    import torch
    s = _scene(d, boxes, m, dense)
    dom, x = B.Domain(s), torch.tensor(s["queries"], dtype=torch.float32, device="cuda")
    Q = len(x)
    x8 = torch.zeros(Q, 8, device="cuda")
    x8[:, :d] = x
    got, work = [], []
    for kw in (dict(full_scan=True), {}, dict(box_test=True), dict(no_box_test=True), dict(wave_scan=True),
               dict(scalar_cull=True)):
        opt = B.options(**kw)
        u, g = torch.empty(Q, device="cuda"), torch.empty(Q, d, device="cuda")
        B.wos_estimate(dom, x, 128, s["sigma"], s["eps"], 5, u, g, opt=opt)
        rec = np.stack([B.wos_debug_walks(dom, s["queries"][q], q, 0, 128, s["sigma"], s["eps"], 5, opt=opt)
                        for q in (0, 3, 6)])
        ub, gb = torch.empty(Q, device="cuda"), torch.empty(Q, 8, device="cuda")
        st = torch.empty(Q, B.BATCH_STATS, dtype=torch.float64, device="cuda")
        # enough walks that a wave carries 64 of them
        B.wos_estimate_batch([dom], x8, [0, Q], [s["sigma"]], [s["eps"]], 25000, 5, ub, gb, st, opt=opt)
        st = st.cpu().numpy()
        got.append((rec, st[:, 9:12], [u, g, ub, gb], st[:, :9]))
        work.append(st[:, 12:])
    for rec, count, out, se in got[1:]:
        assert np.array_equal(rec, got[0][0]) and np.array_equal(count, got[0][1])
        # sums of the same walks, which the kernels' variants may add up in
        # another order: n 2^-53 times the largest term, at most 25000 x 1.1e-16
        # x d / R_0 = 3e-10, then FP32 rounding; standard errors come from a
        # difference of such sums, here a 1e5-th of them or more
        for a, b in zip(out, got[0][2]):
            assert np.allclose(a.cpu().numpy(), b.cpu().numpy(), rtol=2.0 ** -23, atol=1e-9)
        assert np.allclose(se, got[0][3], rtol=1e-6, atol=1e-9)
    full, default, box, no_box, wave, vector = (w[:, 1 if boxes else 0].sum() for w in work)
    # member distances: a pair that fails its box test costs none, a pair scan
    # evaluates no more than the walkers that share a wave, and those no more
    # than a full scan (the bundle alone is most of it)
    assert 0 < box <= no_box <= wave < full and box <= default <= no_box <= vector < full
    assert work[3][:, 3].sum() == 0 < work[2][:, 3].sum()
