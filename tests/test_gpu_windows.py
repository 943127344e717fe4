"""Windows that end at a wall: a tile reaching the right wall is moved left to
end there, so it may start at an odd or unaligned point (rods and the last
waves of a batch's rods)."""
import numpy as np
import pytest

import oracle
from paper_1310_3422_amd import ge, inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# FP64: the bar of the sweep's parity tests.  FP32: u is rounded to half a
# unit (6e-8 of its size) once a level, so 40 levels of rough data stay
# below 40 * 6e-8 = 2.4e-6 of the largest values; 1e-5 leaves room for the
# norm of the result falling as the data smooths.
BARS = {"fp64": 1e-12, "fp32": 1e-5, "fp32c": 1e-5}


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32c"])
@pytest.mark.parametrize("waves", [1, 4])
@pytest.mark.parametrize("extra", [0, 1, 2, 3, 5, 8])
def test_rod_window_ending_at_the_right_wall(precision, waves, extra):
    """Rods of one window and up to a few points more, and of two cores and
    the same: moving walls, a source and the flux, both first parities."""
    tile, depth = 8, 9
    window = 64 * tile * waves
    halo = 10 if precision == "fp64" else 12
    for n in (window + extra, 2 * (window - 2 * halo) + extra):
        w = inputs.moving_wall_rod(n, r=1.5, nsteps=40, step0=1)
        u0 = inputs.sine_rod(n, n) + 0.1 * np.random.default_rng(n).standard_normal(n)
        v0 = ge.unpack_state(ge.pack_state(u0, precision), n, precision)
        dt = ge.state_dtype(precision)
        b = torch.from_numpy(w.src_b).to(dt).cuda()
        d = lambda a: torch.from_numpy(np.asarray(a, dtype=np.float64)).cuda()
        gr = w.g_right + 0.5
        for step0 in (0, 1):
            plan = ge.Plan(n, 1.5, precision, src_b=b, tile=tile, waves=waves, depth=depth)
            u = ge.pack_state(u0, precision)
            flux = torch.zeros(2, dtype=torch.float64, device="cuda")
            plan.step_n(u, step0, 40, g_left_t=d(w.g_left), g_right_t=d(gr), src_a_t=d(w.src_a),
                        flux=flux)
            torch.cuda.synchronize()
            want_flux = np.zeros(2)
            want = oracle.step_n(v0, 1.5, 40, step0=step0, gl=w.g_left, gr=gr,
                                 src_b=b.double().cpu().numpy(), src_a=w.src_a, flux=want_flux)
            got = ge.unpack_state(u, n, precision)
            err = np.linalg.norm(got - want) / np.linalg.norm(want)
            assert err < BARS[precision], (n, step0, err)
            np.testing.assert_allclose(flux.cpu().numpy(), want_flux, rtol=10 * BARS[precision])


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp32c"])
@pytest.mark.parametrize("levels", [2, 7, 40])
def test_batch_last_wave_ending_at_the_right_wall(precision, levels):
    """Every remainder of a rod's length modulo 4, at lengths that take two
    and three overlapping waves: the bits of ge_step_n, first levels of both
    parities, calls with and without a refresh of the shared lanes."""
    n = np.array([base + e for base in (300, 512, 700, 2100) for e in range(4)], dtype=np.int64)
    offsets = np.zeros(n.size + 1, dtype=np.int64)
    offsets[1:] = np.cumsum((n + 3) // 4 * 4)
    rng = np.random.default_rng(levels)
    r, gl, gr = rng.uniform(0.3, 3.0, n.size), rng.uniform(-1, 1, n.size), rng.uniform(-1, 1, n.size)
    u0 = rng.standard_normal(int(offsets[-1]))
    for step0 in (0, 1):
        batch = ge.Batch(n, offsets, r, gl, gr, precision, sync=3)
        u = ge.pack_batch_state(u0, offsets, n, precision)
        batch.solve(u, step0, levels, batch.new_workspace())
        torch.cuda.synchronize()
        got = u.cpu().numpy()
        for i in range(n.size):
            one = ge.pack_state(u0[offsets[i]:offsets[i] + n[i]], precision)
            ge.Plan(int(n[i]), float(r[i]), precision, g_left=gl[i], g_right=gr[i]).step_n(
                one, step0, levels)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(
                ge.unpack_batch_rod(got, offsets, n, i, precision),
                ge.unpack_state(one, int(n[i]), precision), err_msg=str((int(n[i]), step0)))
