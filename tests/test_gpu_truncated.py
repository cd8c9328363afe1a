"""Records of walks that the step cap cuts off: the component they name is the
nearest one at their last point, also where the goal ball is looked up among
the spheres (16 of them or more), as a scan of every obstacle names it."""
import numpy as np
import pytest

from paper_2406_01713_amd import scenes as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [2, 5, 8])
@pytest.mark.parametrize("m", [8, 16, 80])
@pytest.mark.parametrize("fp64", [False, True])
def test_class_of_truncated_walks(d, m, fp64):
    import torch  # noqa: F401  (the HIP runtime the library binds to)
    from paper_2406_01713_amd import binding as B
    s = S.scene_spheres(d, m_sph=m, n_queries=1, sigma=1.0, eps=1e-4)
    s["goal_r"] = 0.3
    x0 = np.asarray(s["goal_c"], float).copy()
    x0[0] -= np.sign(x0[0]) * 0.45  # the goal is near, most walks' nearest component
    dom = B.Domain(s)
    cap = 3
    a, b = (B.wos_debug_walks(dom, x0, 0, 0, 200, 1.0, s["eps"], 17, opt=B.options(fp64, max_steps=cap, full_scan=f))
            for f in (False, True))
    assert np.array_equal(a, b)
    cut = a[:, d + 4] == 2
    assert cut.sum() > 100 and np.all(a[cut, d + 3] == cap)
    assert (a[cut, d + 5] == 0).sum() > 10  # the goal among them
