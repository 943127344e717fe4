"""The host side of batch plans on the CPU, over a stand-in for the HIP runtime
(fake_hip.c): plans for devices with few or no compute units, and the order in
which runs are enqueued."""
import os

import pytest

from hip_stand_in import child
from paper_1310_3422_amd import ge

pytestmark = pytest.mark.skipif(not os.path.exists(ge.LIB_PATH), reason="libge.so not built")

@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return tmp_path_factory.mktemp("hip")


@pytest.mark.parametrize("units", [0, 1, 2, 8, 32, 64, 128, 256, 304])
def test_plans_for_any_number_of_compute_units(fake, units):
    """Every batch gets a plan (without a device, 0 units: an error), whose
    windows cover every rod."""
    out = child(fake, f"""
got = []
for prec in ("fp64", "fp32", "fp32c"):
    for sizes in ([5000], [4465], [300000], [60000] * 8, [768000], [100, 5000], [800000], [4464]):
        fake.fake_reset({units}, -1, 0)
        try:
            b = ge.Batch(*table(sizes), prec)
        except ge.GEError as e:
            got.append([e.status])
            continue
        fake.fake_reset({units}, -1, 0)
        st = ge.lib().ge_solve_batch(b.handle, 1 << 20, 1 << 30, 0, 100, None)
        got.append([st, len(log())])
print(json.dumps(got))
""")
    if units == 0:
        assert all(g[0] in (ge.GE_ERR_NOMEM, ge.GE_ERR_HIP) for g in out), out
    else:
        assert all(g[0] == ge.GE_OK and g[1] >= 1 for g in out), out


def test_two_threads_run_one_plan(fake):
    """Two host threads that run one plan on streams of their own: whatever the
    side stream waits for, the calling thread's stream recorded last, and the
    caller's stream waits for what the side stream recorded last."""
    events = child(fake, """
b = ge.Batch(*table([100, 5000]), "fp32")
fake.fake_reset(256, -1, 300)
st = [None, None]
def run(i):
    st[i] = ge.lib().ge_solve_batch(b.handle, 1 << 20, 1 << 30, 0, 100, (1 + i) << 8)
ts = [threading.Thread(target=run, args=(i,)) for i in range(2)]
for t in ts: t.start()
for t in ts: t.join()
assert st == [0, 0], st
print(json.dumps(log()))
""")
    main = {str(256): 0, str(512): 1}
    last, waits = {}, 0
    for what, stream, event, thread, _, _ in events:
        if what == "record":
            last[event] = (stream, thread)
        elif what == "wait":
            waits += 1
            assert last[event][1] == thread, (event, thread, last[event], events)
            # the side stream waits for the thread's own main stream, and back
            assert (stream in main) != (last[event][0] in main), events
    assert waits == 4, events


@pytest.mark.parametrize("fail_at", range(4))
def test_a_failed_launch_still_joins_the_side_stream(fake, fail_at):
    """A launch that fails after the fork: the error is returned, and the
    caller's stream waits for what the side stream was given."""
    status, events = child(fake, f"""
b = ge.Batch(*table([100, 5000, 3000]), "fp64")
fake.fake_reset(256, {fail_at}, 0)
st = ge.lib().ge_solve_batch(b.handle, 1 << 20, 1 << 30, 0, 100, 256)
print(json.dumps([st, log()]))
""")
    assert status == ge.GE_ERR_HIP, status
    assert any(e[0] == "failed" for e in events), events
    assert events[-1][:2] == ["wait", "256"], events
    joined = [e for e in events if e[0] == "record" and e[2] == events[-1][2]]
    assert len(joined) == 1 and joined[0][1] != "256", events


@pytest.mark.parametrize("sizes", [[100, 5000], [7] * 9, [4464, 4465, 3000, 1], [400000, 500000, 20]])
def test_info_describes_the_form_that_runs(fake, sizes):
    """ntasks and grid are those of the windows: one per rod of up to 4464
    points, the others' windows as many as rod_k and the launches' grids say."""
    info, grids = child(fake, f"""
sizes = {sizes}
b = ge.Batch(*table(sizes), "fp32")
fake.fake_reset(256, -1, 0)
ge.lib().ge_solve_batch(b.handle, 1 << 20, 1 << 30, 0, 1, 256)
i = b.info()
print(json.dumps([[i["ntasks"], i["grid"]], [int(e[4]) for e in log() if e[0] == "launch"]]))
""")
    whole = [n for n in sizes if n <= 4464]
    tiny = sum(n < 256 for n in whole)
    assert info[0] >= len(sizes)
    if len(whole) == len(sizes):
        assert info == [len(sizes), len(sizes) - tiny + (tiny + 3) // 4]
    # a launch's grid is its workgroups rounded up to 8; a pass of one level is
    # followed by one of none
    if len(whole) < len(sizes):
        grids = grids[:-1]
    assert info[1] <= sum(grids) < info[1] + 8 * len(grids), (info, grids)
