"""The compensated pair on rods too short to fill the chip: windows of
overlapping waves give the bits of the tiles (16 points a lane, four waves),
with moving walls, a source and the walls' flux, at lengths where the windows
change: one wave, one window, a last wave that overlaps more, several windows
of each shape, odd lengths."""
import numpy as np
import pytest

from paper_1310_3422_amd import ge

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [256, 257, 511, 700, 1999, 2048, 2049, 5001, 20224, 60001, 262655,
                               599999, 860001])
@pytest.mark.parametrize("moving", [False, True])
def test_pair_windows_give_the_tiles_bits(n, moving):
    assert torch.cuda.is_available()
    levels, step0 = 61, 3
    g = torch.Generator().manual_seed(n)
    u0 = torch.randn(n, dtype=torch.float64, generator=g).numpy()
    b = torch.randn(n, dtype=torch.float32, generator=g).cuda() if moving else None
    t = np.arange(levels + 1) * 0.13
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    kw = {}
    if moving:
        kw = dict(g_left_t=dev(np.sin(t)), g_right_t=dev(np.cos(3 * t) - 0.3),
                  src_a_t=dev(np.exp(-t[:levels])))
    got = []
    for opts in ({}, dict(tile=16, waves=4, depth=24, schedule=1)):
        plan = ge.Plan(n, 1.7, "fp32c", g_left=0.4, g_right=-0.7, src_b=b, **opts)
        u = ge.pack_state(u0, "fp32c")
        flux = torch.tensor([0.25, -0.5], dtype=torch.float64).cuda() if moving else None
        plan.step_n(u, step0, levels, flux=flux, **kw)
        torch.cuda.synchronize()
        got.append((u.cpu().numpy(), None if flux is None else flux.cpu().numpy()))
    o = ge.lib().ge_comp_offset(n)
    (a, fa), (c, fc) = got
    assert np.array_equal(a[:n], c[:n]) and np.array_equal(a[o:o + n], c[o:o + n])
    if moving:
        assert np.array_equal(fa, fc)
