"""Host-side behaviour of the library around its GPU calls, on a stand-in for
the HIP runtime (fake_hip.c: device memory is host memory, kernels do not run,
every launch takes the same time).  Each check runs in a process of its own,
which loads the stand-in before the library."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HEAD = """
import ctypes as C, sys
F = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
F.fake_hip_log.restype = C.c_char_p
F.fake_hip_fail_above.argtypes = [C.c_size_t]
import numpy as np
from paper_2406_01713_amd import binding as B, scenes as S

def launches(name):
    return [tuple(map(int, l.split()[1:])) + (l.split()[0],) for l in F.fake_hip_log().decode().splitlines() if name in l]

def batch(dom, d, Q, n_walks, call="estimate"):
    off, one = np.array([0, Q], dtype=np.int64), np.ones(1)
    q, u = np.zeros((Q, 8), np.float32), np.zeros(Q, np.float32)
    nw = np.array([n_walks], dtype=np.int64)
    i64p, p = C.POINTER(C.c_int64), lambda a: a.ctypes.data_as(C.c_void_p)
    hs = (C.c_void_p * 1)(dom.handle.value)
    if call == "estimate":
        return B.check(B.lib.wos_estimate_batch(hs, 1, p(q), off.ctypes.data_as(i64p), B._dp(one), B._dp(0.01 * one),
                                                nw.ctypes.data_as(i64p), 1, p(u), None, None, None, None, None, None,
                                                None, None))
    r = B.TuneResult()
    B.check(B.lib.wos_autotune_batch(hs, 1, p(q), off.ctypes.data_as(i64p), B._dp(one), B._dp(0.01 * one),
                                     nw.ctypes.data_as(i64p), 1, 0, None, C.byref(r)))
    return r
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("hip") / "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(ROOT, "tests", "fake_hip.c")], check=True)

    def go(code):
        r = subprocess.run([sys.executable, "-c", HEAD + code, so], cwd=ROOT, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr
        return r.stdout
    return go


def test_jac_takes_no_queries(run):
    """No query rows: there is nothing to write, so the (empty) outputs may be
    NULL, as in wos_estimate; with rows the derivatives' array is required."""
    run("""
dom = B.Domain(S.scene_spheres(3, m_sph=8, n_queries=1))
for fp64 in (False, True):
    opt = C.byref(B.options(fp64))
    assert B.lib.wos_estimate(dom.handle, None, 0, 8, 1.0, 1e-3, 1, None, None, None, opt, None) == 0
    assert B.lib.wos_estimate_jac(dom.handle, None, 0, 8, 1.0, 1e-3, 1, None, None, None, None, opt, None) == 0
assert not launches("kernel")
q = np.zeros((1, 3))
p = q.ctypes.data_as(C.c_void_p)
assert B.lib.wos_estimate_jac(dom.handle, p, 1, 8, 1.0, 1e-3, 1, p, None, None, None, None, None) == B.WOS_EINVAL
assert b"out_jac" in B.lib.wos_last_error()
assert B.lib.wos_estimate_jac(dom.handle, p, 1, 8, 1.0, 1e-3, 1, None, None, None, p, None, None) == B.WOS_EINVAL
assert b"out_u" in B.lib.wos_last_error()
""")


@pytest.mark.parametrize("boxes", [False, True])
def test_domain_without_room_for_its_lists(run, boxes):
    """The cell lists only save work: a domain whose lists cannot be allocated
    is made without them (its steps scan clusters); one whose obstacles cannot
    is refused."""
    run(f"""
s = S.scene_spheres(2, m_sph=200, n_queries=1)
if {boxes}:
    s.update(box_c=s["sph_c"], box_h=np.repeat(s["sph_r"][:, None], 2, 1), sph_c=np.zeros((0, 2)), sph_r=np.zeros(0))
dom = B.Domain(s)
batch(dom, 2, 3, 100)
(l,) = launches("persistent_kernel")
assert "persistent_kernelILb0ELb0ELb1E" in l[3], l  # <forward, no source, lists, ...>
F.fake_hip_fail_above(1 << 20)  # 204800 cells take 1.6 MB and more, every other table below 0.1
dom2 = B.Domain(s)
assert F.hipGetLastError() == 0
F.fake_hip_clear()
F.fake_hip_fail_above(0)
batch(dom2, 2, 3, 100)
(l,) = launches("persistent_kernel")
assert "persistent_kernelILb0ELb0ELb0E" in l[3], l  # <forward, no source, no lists, ...>
F.fake_hip_fail_above(256)
try:
    B.Domain(s)
    raise SystemExit("made without its obstacles")
except B.WosError as e:
    assert e.code == -3, e
""")


def test_largest_single_environment_call_is_refused(run):
    """2^32 queries of 2^31 walks, the largest counts the call takes, are 2^63
    walks: more partial sums than there is memory for, refused before any
    launch."""
    run("""
dom = B.Domain(S.scene_spheres(3, m_sph=8, n_queries=1))
F.fake_hip_clear()
F.fake_hip_fail_above(1 << 40)
p = C.c_void_p(8)
for q, n in ((1 << 32, 1 << 31), (1 << 32, 1 << 30), (1 << 31, 1 << 31)):
    assert B.lib.wos_estimate(dom.handle, p, q, n, 1.0, 1e-3, 1, p, None, None, None, None) == -3, (q, n)
assert not launches("plain_kernel"), launches("")
""")


@pytest.mark.parametrize("q,n", [(1, 100), (3, 1000), (1, 100000), (7, 30000), (200, 4096)])
def test_tuner_starts_from_the_untuned_shape(run, q, n):
    """Where every shape takes the same time the tuner keeps the one it started
    from, which is what an untuned call of the batch launches, so ms_default is
    that call's time."""
    run(f"""
dom = B.Domain(S.scene_spheres(3, m_sph=40, n_queries=1))
batch(dom, 3, {q}, {n})
(plain,) = launches("persistent_kernel")
F.fake_hip_clear()
r = batch(dom, 3, {q}, {n}, "tune")
assert launches("persistent_kernel")[0][:3] == plain[:3], (launches("persistent_kernel")[0], plain)
assert r.ms_best == r.ms_default == 1.0
F.fake_hip_clear()
batch(dom, 3, {q}, {n})  # the kept shape
assert launches("persistent_kernel")[0][:3] == plain[:3]
walks = {q} * {n}
want = 8 if walks * 8 <= 163840 else 4 if walks * 4 <= 163840 else 2 if walks * 2 <= 163840 else 1
assert r.lanes_per_walker == want and r.walks_per_lane == (1 if walks <= 262144 else 2), (r.lanes_per_walker, r.walks_per_lane)
assert (r.waves_per_block, r.units_per_wave, r.grid_mult) == (4, 4, 1)
""")
