"""A call's own levels decide the windows it runs in, where the plan leaves them to
the library: checked on the CPU by what is enqueued over a stand-in for the HIP
runtime (fake_hip.c)."""
import os

import pytest

from hip_stand_in import child
from paper_1310_3422_amd import ge

pytestmark = pytest.mark.skipif(not os.path.exists(ge.LIB_PATH), reason="libge.so not built")


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return tmp_path_factory.mktemp("hip")


# points, k, precision, the most levels of a launch in narrow windows, the
# threads of a workgroup of the plan's own shape
@pytest.mark.parametrize("n,k,prec,limit,threads", [
    (1 << 18, 4, "fp32", 32, 256), (1 << 20, 4, "fp64", 24, 256), (1 << 20, 16, "fp64", 24, 256),
    (1 << 15, 2, "fp32", 24, 128), (1 << 22, 8, "fp64", 16, 512), (1 << 24, 8, "fp64", 8, 512),
    (1 << 24, 16, "fp64", 8, 256), (1 << 17, 8, "fp64", 0, 64)])
def test_subdomain_calls_of_few_levels(fake, n, k, prec, limit, threads):
    levels = [1, 2, 8] + ([2 * limit, 2 * limit + 1] if limit else [])
    got = child(fake, f"""
plan = ge.Plan({n - 1}, 1.0, "{prec}", k={k})
out = []
for L in {levels}:
    fake.fake_reset(256, -1, 0)
    st = ge.lib().ge_step_n(plan.handle, 1 << 20, 1 << 40, 0, L, None, None, None, None, None)
    out.append([st, [int(e[5]) for e in log() if e[0] == "launch"]])
print(json.dumps(out))
""")
    for L, (status, blocks) in zip(levels, got):
        assert status == ge.GE_OK
        assert len(blocks) == min(L, 2), (L, blocks)
        want = 64 if (L + 1) // 2 <= limit or (L == 1 and limit) else threads
        assert set(blocks) == {want}, (L, blocks)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("nx,ny", [(4096, 4096), (8192, 1024), (3000, 70)])
def test_grid_calls_of_few_levels(fake, nx, ny, prec):
    """The windows' halo is the call's own levels' (one more point a side, even),
    whatever the levels of the deepest launch would be: as many workgroups as
    windows of some height with that halo, and no copy where an even number of
    launches will do."""
    got = child(fake, f"""
out = []
for L in (1, 2, 3, 5, 8, 200):
    d = ge.ge_2d_desc({nx}, {ny}, 1.0, 1.0, "{prec}")
    fake.fake_reset(256, -1, 0)
    st = ge.lib().ge_2d_step_n(ctypes.byref(d), 1 << 20, 1 << 40, 0, L, None)
    e = log()
    out.append([L, st, [int(x[4]) for x in e if x[0] == "launch"], [x[0] for x in e].count("copy")])
print(json.dumps(out))
""")
    for L, status, groups, copies in got:
        assert status == ge.GE_OK and copies == (L == 1), (L, copies)
        n = len(groups)
        halo = ((L + n - 1) // n + 2) // 2 * 2
        cx = 128 - 2 * halo
        sizes = []
        for rows in (32, 64, 128):
            tiles = -(-nx // cx) * -(-ny // (rows - 2 * halo)) if rows > 2 * halo else 0
            sizes.append((tiles + 7) // 8 * 8)
        assert set(groups) <= set(sizes) and len(set(groups)) == 1, (L, groups, sizes)
        assert n <= 2 or L > 8, (L, n)
