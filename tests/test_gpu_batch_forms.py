"""The two forms of a batch run under replay, capture and threads: the persistent
launch (sync 3, an instantiated graph per state, workspace, parity and level
count), and the split into windows that sync 0 takes."""
import threading

import numpy as np
import pytest

from paper_1310_3422_amd import ge, inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PRECISIONS = ["fp64", "fp32", "fp32c"]


def _batch(sizes, seed, precision, **options):
    n = np.array(sizes, dtype=np.int64)
    offsets = np.zeros(n.size + 1, dtype=np.int64)
    offsets[1:] = np.cumsum((n + 3) // 4 * 4)
    rng = np.random.default_rng(seed)
    table = (n, offsets, rng.uniform(0.3, 3.0, n.size), rng.uniform(-1, 1, n.size),
             rng.uniform(-1, 1, n.size))
    u0 = rng.standard_normal(int(offsets[-1]))
    return ge.Batch(*table, precision, **options), table, u0, \
        ge.pack_batch_state(u0, offsets, n, precision)


def _check_rods(got, table, u0, precision, step0, levels):
    """Every rod of the host copy has the bits of ge_step_n."""
    n, offsets, r, gl, gr = table
    for i in range(n.size):
        one = ge.pack_state(u0[offsets[i]:offsets[i] + n[i]], precision)
        ge.Plan(int(n[i]), float(r[i]), precision, g_left=gl[i], g_right=gr[i]).step_n(
            one, step0, levels)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(ge.unpack_batch_rod(got, offsets, n, i, precision),
                                      ge.unpack_state(one, int(n[i]), precision),
                                      err_msg=str((int(n[i]), step0, levels)))


@pytest.mark.parametrize("precision", PRECISIONS)
def test_persistent_graphs_replay_and_make_room(precision):
    """More keys than the plan keeps graphs, each run twice in turn, so that
    graphs are replayed, replaced and captured again; eager work between."""
    batch, table, u0, start = _batch([7, 300, 5000, 20011], 31, precision, sync=3)
    want = {}
    for rep in range(2):
        for key, (step0, levels) in enumerate([(0, 1), (1, 40), (0, 40), (0, 17), (1, 64), (0, 90)]):
            u, ws = start.clone(), batch.new_workspace()
            for again in range(2):
                u.copy_(start)
                float(torch.randn(1 << 16, device="cuda").sum())
                batch.solve(u, step0, levels, ws)
                batch.check()
                got = u.cpu().numpy()
                if key not in want:
                    want[key] = got
                    _check_rods(got, table, u0, precision, step0, levels)
                np.testing.assert_array_equal(got, want[key], err_msg=str((rep, key, again)))


@pytest.mark.parametrize("precision", PRECISIONS)
def test_persistent_long_rods(precision):
    """Rods above the on-chip limit beside short ones, below, at and above one
    pass, even and odd level counts, from both parities."""
    cap = 65536 if precision == "fp32" else 32768
    batch, table, u0, start = _batch([cap + 1, cap + 1000, 2 * cap + 77, 100, cap, 1], 32,
                                     precision, sync=3)
    ws = batch.new_workspace()
    for step0, levels in ((0, 1), (1, 2), (1, 33), (0, 64), (3, 131)):
        u = start.clone()
        batch.solve(u, step0, levels, ws)
        batch.check()
        _check_rods(u.cpu().numpy(), table, u0, precision, step0, levels)


def test_persistent_tuned_plan(tmp_path, monkeypatch):
    monkeypatch.setenv("GE_TUNE_CACHE", str(tmp_path / "tune.txt"))
    rb = inputs.rod_batch(seed=33, nrods=24, nmin=256, nmax=65536, align=4)
    got = []
    for tune in (False, True):
        b = ge.Batch.from_inputs(rb, "fp32", tune=tune, sync=3)
        u = ge.pack_batch_state(rb.u0, rb.offsets, rb.n, "fp32")
        b.solve(u, 0, 30, b.new_workspace())
        b.check()
        got.append(u.cpu().numpy())
    np.testing.assert_array_equal(got[0], got[1])


@pytest.mark.parametrize("precision", PRECISIONS)
def test_windows_captured_in_a_graph(precision):
    """A run whose short rods go to the plan's side stream beside the passes,
    captured on a side stream of the caller's and replayed."""
    batch, table, u0, start = _batch([7, 300, 3000, 5000, 20011, 100001], 34, precision)
    ws = batch.new_workspace()
    want = start.clone()
    batch.solve(want, 0, 90, ws)
    batch.check()
    u, stream = start.clone(), torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        batch.solve(u, 0, 90, ws, stream=stream)
    for rep in range(4):
        u.copy_(start)
        graph.replay()
        float(torch.randn(1 << 16, device="cuda").sum())
        torch.cuda.synchronize()
        assert torch.equal(u, want), rep
    batch.check()


@pytest.mark.parametrize("precision", PRECISIONS)
def test_two_threads_run_one_plan(precision):
    batch, table, u0, start = _batch([7, 300, 3000, 5000, 20011], 35, precision)
    want = start.clone()
    batch.solve(want, 0, 90, batch.new_workspace())
    torch.cuda.synchronize()
    bufs = [(start.clone(), batch.new_workspace(), torch.cuda.Stream()) for _ in range(2)]
    for u, _, _ in bufs:
        u.copy_(start)
    torch.cuda.synchronize()
    errors = []

    def run(u, ws, stream):
        try:
            for _ in range(6):
                batch.solve(u, 0, 90, ws, stream=stream)
        except Exception as e:          # shown by the thread that joins
            errors.append(e)

    threads = [threading.Thread(target=run, args=b) for b in bufs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors
    for _ in range(5):
        batch.solve(want, 0, 90, bufs[0][1])
    torch.cuda.synchronize()
    for u, _, _ in bufs:
        assert torch.equal(u, want)
