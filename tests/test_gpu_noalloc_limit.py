"""The no-allocation batch near the limit of its array: a batch of 5-D and
smaller environments runs five waves per SIMD and would be cut into a quarter
more work units than four waves ask for; where those outgrow the array the
call takes the shorter list of units.  The walks are the same, only the
grouping of the FP64 sums differs, so each FP32 result may differ from the
allocating call's by its final rounding."""
import numpy as np
import pytest

from paper_2406_01713_amd import scenes as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [3, 5])
def test_batch_that_fits_only_in_longer_units(d):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2406_01713_amd import binding as B
    s = S.with_bdata(S.scene_spheres(d, n_queries=1, n_walks=10, seed=1), 2,
                     ak=S.plane_wave_k(d, S.scene_spheres(d, n_queries=1, n_walks=10, seed=1)["sigma"], seed=3))
    # 310000 one-unit queries and one query of 7e6 walks (10.1e6 walks): ranges
    # of 512 walks for 20480 units (323672 rows, 208 bytes each, more than 64
    # MiB), of 640 for 16384 (320938 rows, which fit)
    n = 310001
    q = torch.zeros(n, 8, device="cuda")
    q[:, :d] = torch.as_tensor(s["queries"][0], dtype=torch.float32, device="cuda")
    off = np.array([0, n - 1, n], dtype=np.int64)
    dom = B.Domain(s)
    out = []
    for noalloc in (True, False):
        u = torch.full((n,), float("nan"), device="cuda")
        B.wos_estimate_batch([dom, dom], q, off, [s["sigma"]] * 2, [s["eps"]] * 2, [10, 7000000], 1, u, noalloc=noalloc)
        torch.cuda.synchronize()
        out.append(u.cpu().numpy().astype(np.float64))
    assert np.all(np.isfinite(out[0])) and np.any(out[0] != 0)
    # sums of 10 walks are one unit in both: bitwise; the long query: one FP32 ulp
    assert np.array_equal(out[0][:-1], out[1][:-1])
    assert abs(out[0][-1] - out[1][-1]) <= 2.0 ** -23 * abs(out[1][-1])
