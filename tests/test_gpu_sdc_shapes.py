"""The windows that the library chooses for the sub-domain scheme, at the
lengths where the choice changes: the same bits as single-wave windows of 20
levels, launched per tile (the tiling never enters the arithmetic), over a
run that is no multiple of any depth."""
import numpy as np
import pytest

from paper_1310_3422_amd import ge

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def couples(k, waves, depth, launch_waves):
    """the most couples that windows of `waves` waves take in launch_waves"""
    halo = (depth * (k + 1) + 2 + 2 * k - 1) // (2 * k)
    return (64 * waves - 2 * halo) * (launch_waves // waves)


# precision, k, couples of the last rod before the change of shape, the shape there
# and right after
EDGES = [
    ("fp64", 2, 64, (1, 20), (2, 64)),
    ("fp32", 8, 64, (1, 20), (1, 32)),
    ("fp32", 16, couples(16, 1, 32, 1024), (1, 20), (4, 64)),
    ("fp64", 16, couples(16, 1, 32, 1024), (1, 24), (4, 64)),
    ("fp64", 2, couples(2, 2, 64, 1024), (2, 64), (4, 64)),
    ("fp32", 4, couples(4, 1, 32, 1024), (1, 32), (4, 64)),
    ("fp64", 8, couples(8, 1, 32, 1024), (1, 32), (4, 64)),
    ("fp64", 16, couples(16, 4, 64, 2048), (4, 64), (1, 24)),
    ("fp32", 16, couples(16, 4, 64, 4096), (4, 64), (8, 96)),
    ("fp32", 2, couples(2, 4, 64, 4096), (4, 64), (8, 64)),
]


@pytest.mark.parametrize("precision,k,last,before,after", EDGES)
def test_chosen_windows_give_the_same_bits(precision, k, last, before, after):
    assert torch.cuda.is_available()
    for nsdc, shape in ((last, before), (last + 1, after)):
        n = 2 * k * nsdc - 1
        g = torch.Generator().manual_seed(nsdc)
        u0 = torch.randn(n, dtype=torch.float64, generator=g).to(ge.state_dtype(precision)).cuda()
        plan = ge.Plan(n, 2.3, precision, g_left=0.4, g_right=-0.25, k=k)
        ref = ge.Plan(n, 2.3, precision, g_left=0.4, g_right=-0.25, k=k, schedule=1, waves=1,
                      depth=20)
        c = plan.config()
        assert (c["waves"], c["depth"]) == shape
        a, b = u0.clone(), u0.clone()
        plan.step_n(a, 1, 101)
        ref.step_n(b, 1, 101)
        torch.cuda.synchronize()
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy()), (precision, k, nsdc)
