"""The library's split of a batch into windows: rods at the edges of every kind
(one wave, a block window of each shape, block and single-wave windows of a
pass) get the bits of ge_step_n, beside each other and alone."""
import numpy as np
import pytest

from paper_1310_3422_amd import ge

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EDGES = [1, 2, 3, 63, 64, 65, 255, 256, 257, 880, 881, 1392, 1393, 1904, 1905, 2928, 2929, 4464]
SMALL = EDGES + [4465, 6000, 9001]                    # longer rods: block windows
LARGE = [300, 4465, 65537, 100001, 250000, 400003]     # single-wave windows, 16 points a lane


def _batch(sizes, seed):
    n = np.array(sizes, dtype=np.int64)
    offsets = np.zeros(n.size + 1, dtype=np.int64)
    offsets[1:] = np.cumsum((n + 3) // 4 * 4)
    rng = np.random.default_rng(seed)
    return (n, offsets, rng.uniform(0.3, 3.0, n.size), rng.uniform(-1, 1, n.size),
            rng.uniform(-1, 1, n.size), rng.standard_normal(int(offsets[-1])))


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32c"])
@pytest.mark.parametrize("name,sizes", [("edges", EDGES), ("small", SMALL), ("large", LARGE),
                                        ("one", [5000]), ("tiny", [7])])
def test_windows_give_the_bits_of_single_rods(name, sizes, precision):
    n, offsets, r, gl, gr, u0 = _batch(sizes, len(sizes))
    batch = ge.Batch(n, offsets, r, gl, gr, precision)
    ws = batch.new_workspace()
    start = ge.pack_batch_state(u0, offsets, n, precision)
    for step0, levels in ((0, 1), (1, 2), (1, 50), (0, 131)):
        u = start.clone()
        batch.solve(u, step0, levels, ws)
        batch.check()
        got = u.cpu().numpy()
        for i in range(n.size):
            one = ge.pack_state(u0[offsets[i]:offsets[i] + n[i]], precision)
            ge.Plan(int(n[i]), float(r[i]), precision, g_left=gl[i], g_right=gr[i]).step_n(
                one, step0, levels)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(ge.unpack_batch_rod(got, offsets, n, i, precision),
                                          ge.unpack_state(one, int(n[i]), precision),
                                          err_msg=str((int(n[i]), step0, levels)))
        # the values between the rods are left alone
        gap = np.ones(got.size, dtype=bool)
        for i in range(n.size):
            gap[offsets[i]:offsets[i] + n[i]] = False
            if precision == "fp32c":
                e = int(ge.lib().ge_comp_offset(int(offsets[-1]))) + offsets[i]
                gap[e:e + n[i]] = False
        np.testing.assert_array_equal(got[gap], start.cpu().numpy()[gap])


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32c"])
def test_replays_and_two_streams(precision):
    """The captured branches replay with eager work between them, and two runs
    of one plan on two streams, each with its own workspace, do not meet."""
    n, offsets, r, gl, gr, u0 = _batch(SMALL + [70000], 5)
    batch = ge.Batch(n, offsets, r, gl, gr, precision)
    start = ge.pack_batch_state(u0, offsets, n, precision)
    ref = start.clone()
    batch.solve(ref, 0, 90, batch.new_workspace())
    torch.cuda.synchronize()
    bufs = [(start.clone(), batch.new_workspace(), torch.cuda.Stream()) for _ in range(2)]
    torch.cuda.synchronize()
    for rep in range(3):
        for u, ws, st in bufs:
            with torch.cuda.stream(st):
                u.copy_(start)
                batch.solve(u, 0, 90, ws, stream=st)
        float(torch.randn(1 << 16, device="cuda").sum())
        torch.cuda.synchronize()
        for u, _, _ in bufs:
            assert torch.equal(u, ref), rep
