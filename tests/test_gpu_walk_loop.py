"""The walk loop around a work unit: records of finished walks queued and added
up (queues of fewer than 64 entries, many walks ending in one step), ranges of
one query's walks, the point source's Green's function in every dimension."""
import numpy as np
import pytest

from paper_2406_01713_amd import scenes as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch  # noqa: F401  (the HIP runtime the library binds to)
    from paper_2406_01713_amd import binding
    return binding


@pytest.fixture(scope="module")
def oracle():
    from oracle import oracle as O
    O.build()
    return O


@pytest.mark.parametrize("d", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("sigma", [0.0, 3.0])
@pytest.mark.parametrize("fp64", [False, True])
def test_source_terms_in_every_dimension(B, oracle, d, sigma, fp64):
    """Walks from points whose first ball holds the source, and from points
    whose walks meet it later, against the oracle's, walk by walk.  FP64: both
    sides round G_B (a difference of terms that agree to a few digits near the
    ball's edge) and d u / d sigma to about 1e-13 of their parts; 1e-8 is far
    above.  FP32: the walk's drift, 2e-4 for 95 % of the walks."""
    q = np.zeros((2, d))
    q[0, 0], q[1, -1] = 0.2, 0.7
    s = S.scene_ball_source(d, sigma=sigma, queries=q, n_walks=64, seed=3)
    dom, odom = B.Domain(s), oracle.Domain(s)
    same = close = 0
    for qi in range(2):
        rec = B.wos_debug_walks(dom, q[qi], qi, 0, 64, sigma, s["eps"], 3, B.options(fp64))
        for w in range(64):
            r = oracle.walk(s, q[qi].astype(np.float64 if fp64 else np.float32).astype(np.float64), w, qi, seed=3, dom=odom)
            if int(rec[w, d + 3]) != r["steps"]:
                continue
            same += 1
            tol = 1e-8 if fp64 else 2e-4
            close += abs(rec[w, 0] - r["u"]) <= tol * max(1.0, abs(r["u"])) and \
                np.allclose(rec[w, 1:1 + d], r["grad"], rtol=tol, atol=tol * max(1.0, np.abs(r["grad"]).max()))
    assert same >= (126 if fp64 else 120), same
    assert close >= (same if fp64 else 0.95 * same), (close, same)


@pytest.mark.parametrize("d,src", [(2, False), (8, False), (8, True)])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 300, 4097])
def test_many_walks_end_in_one_step(B, d, src, n):
    """A step cap ends whole waves at once, more walks than the record queue
    holds (42 and fewer in 8-D): the estimate, the batched call and the walk
    records count and sum the same walks."""
    import torch
    s = S.scene_spheres(d, m_sph=40, n_queries=2, n_walks=n, sigma=1.0, eps=1e-3)
    s["bdata"] = dict(s["bdata"], g_outer=1.0)
    if src:
        s = S.with_source(s, s["queries"][0] + 0.05, keep_goal=True)
    dom = B.Domain(s)
    opt = B.options(max_steps=6)
    rec = [B.wos_debug_walks(dom, q, i, 0, n, 1.0, 1e-3, 9, opt) for i, q in enumerate(np.float32(s["queries"]).astype(float))]
    x = torch.tensor(s["queries"], dtype=torch.float32, device="cuda")
    u, g = torch.empty(2, device="cuda"), torch.empty(2, d, device="cuda")
    st = torch.empty(2, d + 4, dtype=torch.float64, device="cuda")
    B.wos_estimate(dom, x, n, 1.0, 1e-3, 9, u, g, st, opt=opt)
    q8 = torch.zeros(2, 8, device="cuda")
    q8[:, :d] = x
    ub, gb = torch.empty(2, device="cuda"), torch.empty(2, 8, device="cuda")
    sb = torch.empty(2, B.BATCH_STATS, dtype=torch.float64, device="cuda")
    B.wos_estimate_batch([dom], q8, [0, 2], [1.0], [1e-3], n, 9, ub, gb, sb, opt=opt)
    u, g, st, ub, gb, sb = [t.cpu().numpy() for t in (u, g, st, ub, gb, sb)]
    for i in range(2):
        m = rec[i].mean(axis=0)
        cut, deg = (rec[i][:, d + 4] == 2).sum(), (rec[i][:, d + 4] == 1).sum()
        assert st[i, d + 1] == m[d + 3] and st[i, d + 2] == cut and st[i, d + 3] == deg
        assert sb[i, 9] == m[d + 3] and sb[i, 10] == cut and sb[i, 11] == deg
        # means of FP64 sums, rounded to FP32
        for got_u, got_g in ((u[i], g[i]), (ub[i], gb[i, :d])):
            assert abs(got_u - m[0]) <= 1e-7 * np.abs(rec[i][:, 0]).mean()
            assert np.allclose(got_g, m[1:1 + d], rtol=1e-7, atol=1e-7 * np.abs(rec[i][:, 1:1 + d]).mean())
    assert n < 60 or any((r[:, d + 4] == 2).sum() > 50 for r in rec) or d == 2


def test_ranges_of_one_query_cover_its_walks(B):
    """One query's walks split over many waves, the last range short: the same
    walks as the records, each once (sums of the records to FP64 rounding)."""
    import torch
    n = 300001
    s = S.scene_spheres(2, m_sph=20, n_queries=1, n_walks=n, sigma=0.5, eps=1e-2)
    s["bdata"] = dict(s["bdata"], g_outer=0.5)
    dom = B.Domain(s)
    x = torch.tensor(s["queries"], dtype=torch.float64, device="cuda")
    u, g = torch.empty(1, dtype=torch.float64, device="cuda"), torch.empty(1, 2, dtype=torch.float64, device="cuda")
    st = torch.empty(1, 6, dtype=torch.float64, device="cuda")
    B.wos_estimate(dom, x, n, 0.5, 1e-2, 4, u, g, st, opt=B.options(True))
    r = B.wos_debug_walks(dom, s["queries"][0], 0, 0, n, 0.5, 1e-2, 4, B.options(True))
    assert st[0, 3].item() == r[:, 5].mean()
    # pairwise against chunked FP64 sums of 3e5 values of order 1: 1e-12
    assert abs(u.item() - r[:, 0].mean()) <= 1e-12
    assert np.allclose(g.cpu().numpy()[0], r[:, 1:3].mean(0), rtol=0, atol=1e-11)
