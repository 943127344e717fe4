"""The 2D extension where its windows (128 columns by 32, 64 or 128 rows) meet
the walls: grids smaller than a window in one or both directions, of exactly
one window, and larger ones whose last window starts at an odd row or column."""
import numpy as np
import pytest

import oracle
from paper_1310_3422_amd import ge

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 5), (127, 31), (128, 32), (129, 33), (126, 40), (61, 200),
                                   (200, 30), (128, 64), (237, 65), (131, 131), (255, 258), (530, 129)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_windows_at_the_walls(nx, ny, precision):
    rng = np.random.default_rng([nx, ny])
    u0 = rng.standard_normal((ny, nx))
    u0 = ge.unpack_state(ge.pack_state(u0.ravel(), precision), nx * ny, precision).reshape(ny, nx)
    walls = (0.4, -0.7, 1.1, -0.2)
    # FP32: half a unit (6e-8) per direction and level, 2 x 27 of them at most
    # 3.2e-6 of the largest values; the walls keep the result's norm up
    bar = 1e-12 if precision == "fp64" else 1e-5
    for step0 in (0, 1):
        want = oracle.step2d_n(u0, 1.7, 0.6, 27, step0=step0, walls=walls)
        outs = []
        for depth in (0, 1, 4):
            u = ge.pack_state(u0.ravel(), precision)
            ge.step2d_n(u, nx, ny, 1.7, 0.6, step0, 27, precision, walls, depth=depth)
            torch.cuda.synchronize()
            outs.append(ge.unpack_state(u, nx * ny, precision))
        np.testing.assert_array_equal(outs[1], outs[0])
        np.testing.assert_array_equal(outs[2], outs[0])
        err = np.linalg.norm(outs[0] - want.ravel()) / np.linalg.norm(want)
        assert err < bar, (step0, err)
