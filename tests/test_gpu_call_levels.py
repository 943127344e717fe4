"""Calls of few levels, which run in windows of their own, give the bits of
windows laid out for one number of levels."""
import pytest

from paper_1310_3422_amd import ge

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision,k,nsdc", [("fp64", 2, 8000), ("fp32", 4, 32768),
                                              ("fp64", 8, 100003), ("fp64", 16, 32771),
                                              ("fp32", 16, 262144)])
def test_subdomain_calls(precision, k, nsdc):
    n = 2 * k * nsdc - 1
    g = torch.Generator().manual_seed(nsdc)
    u0 = torch.randn(n, dtype=torch.float64, generator=g).to(ge.state_dtype(precision)).cuda()
    plan = ge.Plan(n, 2.3, precision, g_left=0.4, g_right=-0.25, k=k)
    ref = ge.Plan(n, 2.3, precision, g_left=0.4, g_right=-0.25, k=k, schedule=1, waves=1, depth=20)
    ws = plan.new_workspace()
    for step0, levels in ((0, 1), (1, 2), (1, 3), (0, 16), (1, 17), (0, 33), (1, 48), (0, 49),
                          (0, 64), (1, 65)):
        a, b = u0.clone(), u0.clone()
        plan.step_n(a, step0, levels, workspace=ws)
        ref.step_n(b, step0, levels)
        assert torch.equal(a, b), (step0, levels)
