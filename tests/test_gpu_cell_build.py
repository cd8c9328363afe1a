"""The build of the cell lists where its ways part: tables of ragged tiles in
every dimension, lists longer than the room first made for them, more obstacles
about a wave's cells or a block's tile than they keep apart (1024, 3072).  The
lists show in the walks: bitwise those of a scan of every obstacle."""
import numpy as np
import pytest

from paper_2406_01713_amd import scenes as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    import torch  # noqa: F401  (the HIP runtime the library binds to)
    from paper_2406_01713_amd import binding
    return binding


def _scene(d, c, r, half, boxes=False, geom_d=0, seed=0):
    rng = np.random.default_rng(seed)
    s = S._empty(d)
    if boxes:
        s.update(box_c=c, box_h=np.repeat(r[:, None], d, 1) * rng.uniform(0.3, 1.0, size=(len(r), d)))
    else:
        s.update(sph_c=c, sph_r=r)
    s.update(d=d, goal_c=None, goal_r=None, outer={"kind": "box", "lo": -half, "hi": half},
             bdata=S._bdata(0, d, g_goal=0.0, g_obs=1.0, g_outer=0.25), sigma=0.5, eps=1e-3 * float(half.min()), seed=3)
    if geom_d:
        s["geom_d"] = geom_d
    s["queries"] = rng.uniform(-0.9, 0.9, size=(5, d)) * half
    # two of them next to an obstacle, so that walks end there in any dimension
    for q in (3, 4):
        v = rng.normal(size=d)
        s["queries"][q] = c[q] + 1.02 * r[q] * np.sqrt(d if boxes else 1) * v / np.linalg.norm(v)
    return s


def _check(B, s):
    dom = B.Domain(s)
    hit = 0
    for fp64 in (False, True):
        for i, q in enumerate(s["queries"]):
            a, b = (B.wos_debug_walks(dom, q, i, 0, 128, s["sigma"], s["eps"], 3, opt=B.options(fp64, full_scan=f))
                    for f in (False, True))
            assert np.array_equal(a, b), (fp64, i)
            hit += int(((a[:, s["d"] + 5] == 1) | (a[:, s["d"] + 5] == 2)).sum())
    assert hit > 0  # walks end on obstacles


@pytest.mark.parametrize("d,geom_d", [(2, 1), (2, 0), (3, 0), (4, 0), (5, 0), (6, 0), (7, 0), (8, 0), (8, 5)])
@pytest.mark.parametrize("m", [16, 130])
@pytest.mark.parametrize("boxes", [False, True])
def test_ragged_tables(B, d, geom_d, m, boxes):
    if boxes and geom_d:
        pytest.skip("boxes are never extruded")
    rng = np.random.default_rng(d * 1000 + m)
    half = rng.uniform(1.2, 2.5, size=d)
    _check(B, _scene(d, rng.uniform(-0.9, 0.9, size=(m, d)) * half, rng.uniform(0.05, 0.13 * d, size=m), half, boxes, geom_d))


@pytest.mark.parametrize("m", [600, 1800])
def test_more_entries_than_room(B, m):
    """Points on a circle are about equally near to the cells around its centre:
    these list them all (1800: more than a wave keeps apart), and the table has
    more entries than uniform scenes of that size."""
    t = np.linspace(0, 2 * np.pi, m, endpoint=False)
    s = _scene(2, 0.5 * np.stack([np.cos(t), np.sin(t)], 1), np.zeros(m), np.full(2, 2.0))
    s["queries"][0] = 0.0
    _check(B, s)


@pytest.mark.parametrize("d,boxes", [(2, False), (3, False), (3, True)])
def test_crowded_tiles(B, d, boxes):
    """9000 small obstacles in about a tile's width: none of its cells lists more
    than a header counts, but block and waves go through all of them."""
    rng = np.random.default_rng(7)
    width = 8 * 4.0 / 512 if d == 2 else 4 * 4.0 / 64  # 2^18 cells over [-2, 2]^d
    c = rng.uniform(0.0, width, size=(9000, d))
    c = np.concatenate([c, rng.uniform(-1.9, 1.9, size=(100, d))])
    r = np.concatenate([np.full(9000, 1e-4), np.full(100, 0.05)])
    s = _scene(d, c, r, np.full(d, 2.0), boxes)
    s["queries"][:3] = -0.05 + rng.uniform(-0.02, 0.02, size=(3, d))
    s["eps"] = 1e-4
    _check(B, s)


def test_less_entries_than_room(B):
    """12000 spheres in a slab along one face of a 6-D box: far fewer entries than
    in a uniform scene, so the table is built again to their size."""
    import torch
    d, m = 6, 12000
    rng = np.random.default_rng(11)
    c = rng.uniform(-1.9, 1.9, size=(m, d))
    c[:, 0] = rng.uniform(1.85, 1.95, size=m)
    s = _scene(d, c, rng.uniform(0.01, 0.03, size=m), np.full(d, 2.0))
    _check(B, s)
    torch.zeros(1, device="cuda")
    free = torch.cuda.mem_get_info()[0]
    doms = [B.Domain(s) for _ in range(4)]
    # uniform: 1.8e7 entries guessed, 73 MB; the clusters' tables take 4 MB
    assert (free - torch.cuda.mem_get_info()[0]) / len(doms) < 50e6
