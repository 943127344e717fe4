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
