"""The no-allocation batch near the limit of its array: a batch of 5-D and
smaller environments runs five waves per SIMD and would be cut into a quarter
more work units than four waves ask for, and ranges of equal steps cut a 7-D
query among 3-D ones into more than ranges of equal walks; where those outgrow
the array the call takes the shorter list of units.  The walks are the same, only the
grouping of the FP64 sums differs, so each FP32 result may differ from the
allocating call's by its final rounding."""
import numpy as np
import pytest

from paper_2406_01713_amd import scenes as S

pytestmark = pytest.mark.gpu


# 310000 one-unit queries of 10 walks and one long query: units in the usual
# cut and in the shortest, where the 64 MiB array holds 322624 rows of 208 bytes
@pytest.mark.parametrize("d,d_long,n_long", [
    (3, 3, 7000000),   # 20480 ranges of 512 walks: 323672; 16384 of 640: 320938
    (5, 5, 7000000),
    (3, 7, 5000000),   # 7-D ranges of 384 walks: 323021; equal walks, 512: 319766
])
def test_batch_that_fits_only_in_longer_units(d, d_long, n_long):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2406_01713_amd import binding as B
    n = 310001
    off = np.array([0, n - 1, n], dtype=np.int64)
    q = torch.zeros(n, 8, device="cuda")
    env = []
    for e, k in enumerate((d, d_long)):
        s = S.scene_spheres(k, n_queries=1, n_walks=10, seed=1)
        env.append(S.with_bdata(s, 2, ak=S.plane_wave_k(k, s["sigma"], seed=3)))
        q[off[e]:off[e + 1], :k] = torch.as_tensor(s["queries"][0], dtype=torch.float32, device="cuda")
    doms = [B.Domain(s) for s in env]
    out = []
    for noalloc in (True, False):
        u = torch.full((n,), float("nan"), device="cuda")
        B.wos_estimate_batch(doms, q, off, [s["sigma"] for s in env], [s["eps"] for s in env], [10, n_long], 1, u,
                             noalloc=noalloc)
        torch.cuda.synchronize()
        out.append(u.cpu().numpy().astype(np.float64))
    assert np.all(np.isfinite(out[0])) and np.any(out[0] != 0)
    # sums of 10 walks are one unit in both: bitwise; the long query: one FP32 ulp
    assert np.array_equal(out[0][:-1], out[1][:-1])
    assert abs(out[0][-1] - out[1][-1]) <= 2.0 ** -23 * abs(out[1][-1])
