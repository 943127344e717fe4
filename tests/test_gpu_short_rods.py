"""Rods too short to fill the chip: the library's windows of overlapping waves
give the bits of the tiled sweep at every length where their split changes."""
import numpy as np
import pytest

import oracle
from paper_1310_3422_amd import ge, inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _run(u0, r, step0, levels, precision, w, src, flux, **cfg):
    n = len(u0)
    dt = ge.state_dtype(precision)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()
    b = dev(w.src_b).to(dt) if src else None
    plan = ge.Plan(n, r, precision, g_left=0.3, g_right=-0.2, src_b=b, **cfg)
    u, fl = ge.pack_state(u0, precision), torch.zeros(2, dtype=torch.float64, device="cuda")
    plan.step_n(u, step0, levels, g_left_t=dev(w.g_left) if src else None,
                g_right_t=dev(w.g_right - 0.2) if src else None,
                src_a_t=dev(w.src_a) if src else None, flux=fl if flux else None)
    torch.cuda.synchronize()
    return ge.unpack_state(u, n, precision), fl.cpu().numpy(), plan.config()


# below the smallest window; one wave; two waves by a point; the capacities of
# the shapes (880, 1392, 1904) and of one window (2048); several windows of
# every shape, short last cores; the longest such rod and one more
@pytest.mark.parametrize("n", [1, 2, 3, 63, 255, 256, 257, 463, 464, 465, 880, 881, 1392, 1393, 1905,
                               2047, 2048, 2049, 2050, 4099, 5121, 60001, 150001, 262655, 600003,
                               768000, 768001])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_library_choice_gives_the_bits_of_tiles(n, precision):
    rng = np.random.default_rng(n)
    levels = 61 if n > 10000 else 150
    w = inputs.moving_wall_rod(n, r=2.5, nsteps=levels, step0=1)
    u0 = inputs.sine_rod(n, n) + 0.05 * rng.standard_normal(n)
    for step0, src in ((0, False), (1, True), (1, False)):
        got, fl, cfg = _run(u0, 2.5, step0, levels, precision, w, src, True)
        want, wfl, _ = _run(u0, 2.5, step0, levels, precision, w, src, True, tile=16, waves=4,
                            depth=13)
        np.testing.assert_array_equal(got, want, err_msg=str((cfg, step0, src)))
        np.testing.assert_array_equal(fl, wfl)


@pytest.mark.parametrize("levels", [1, 22, 23, 24, 46, 47, 900])
def test_refreshes_and_launches(levels):
    """Level counts around a refresh (every 23 levels) and several launches,
    one and many windows, against the oracle."""
    for n, r in ((1000, 1.3), (3001, 0.6)):
        u0 = inputs.sine_rod(n, 4) + 0.1 * np.random.default_rng(n).standard_normal(n)
        u, plan = ge.pack_state(u0, "fp64"), ge.Plan(n, r, "fp64", g_left=0.2, g_right=-0.4)
        plan.step_n(u, 3, levels)
        torch.cuda.synchronize()
        want = oracle.step_n(u0, r, levels, step0=3, gl=0.2, gr=-0.4)
        got = ge.unpack_state(u, n, "fp64")
        assert np.linalg.norm(got - want) < 1e-12 * np.linalg.norm(want)


def test_one_window_needs_no_workspace():
    """Rods of up to 2048 points (4096 for the pair) are advanced in place."""
    lib = ge.lib()
    for precision, n in (("fp64", 2048), ("fp32", 2048), ("fp64", 200), ("fp32c", 4096)):
        plan = ge.Plan(n, 1.0, precision)
        u0 = inputs.sine_rod(n, 1)
        u = ge.pack_state(u0, precision)
        st = lib.ge_step_n(plan.handle, ge._ptr(u), None, 0, 50, None, None, None, None,
                           ge._stream_ptr(None))
        assert st == ge.GE_OK, ge.last_error()
        torch.cuda.synchronize()
        v0 = ge.unpack_state(ge.pack_state(u0, precision), n, precision)
        want = oracle.step_n(v0, 1.0, 50)
        err = np.linalg.norm(ge.unpack_state(u, n, precision) - want) / np.linalg.norm(want)
        assert err < (1e-12 if precision == "fp64" else 1e-5)
