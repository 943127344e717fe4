"""FP32 levels round the increment before they add it: rods and batches give the
bits of u + fl(c1 D + fl(c2 D_q)), grids those of u + fl(c2 D_q + fl(c1 D))
(numpy, each FMA rounded once), also where c1 and c2 are dyadic or thirds and
the exact increment often lies half way between two values."""
import numpy as np
import pytest

from paper_1310_3422_amd import ge

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F = np.float32
R = [0.25, 0.5, 1.0, 2.0, 4.0, 1.37]


def _fma(a, b, c):
    """One rounding to FP32 (the product is exact in 64 bits of significand)."""
    return (np.longdouble(a) * np.asarray(b, np.longdouble) + np.asarray(c, np.longdouble)).astype(F)


def _level(u, r, p, gl, gr, src=None, grid=False):
    """One level along the last axis; src: (a, b, tau)."""
    n = u.shape[-1]
    c1, c2, cs = F((r + r * r) / (1 + 2 * r)), F(r * r / (1 + 2 * r)), F(r / (1 + r))
    pad = [(0, 0)] * (u.ndim - 1) + [(1, 1)]
    U = np.pad(u, pad)
    U[..., 0], U[..., -1] = F(gl), F(gr)
    d = U[..., 1:] - U[..., :-1]
    D = d[..., 1:] - d[..., :-1]
    i = np.arange(n)
    q = np.where((i + p) % 2 == 0, i + 1, i - 1)
    alone = (q < 0) | (q >= n)
    qc = np.clip(q, 0, n - 1)
    Dq = D[..., qc]
    inc = np.where(alone, cs * D, _fma(c2, Dq, c1 * D) if grid else _fma(c1, D, c2 * Dq))
    if src is not None:
        a, b, tau = src
        e1, e2, es = F(tau * (1 + r) / (1 + 2 * r)), F(tau * r / (1 + 2 * r)), F(tau / (1 + r))
        inc = _fma(F(a), np.where(alone, es * b, _fma(e1, b, e2 * b[qc])), inc)
    return u + inc.astype(F)


def _rod(u, r, levels, gl, gr):
    for m in range(levels):
        u = _level(u, r, m & 1, gl, gr)
    return u


def _data(n, seed):
    rng = np.random.default_rng(seed)
    x = np.arange(1, n + 1) / (n + 1)
    gl, gr = (float(F(v)) for v in rng.uniform(-1, 1, 2))
    return (gl + (gr - gl) * x + np.sin(np.pi * x)).astype(F), gl, gr


@pytest.mark.parametrize("r", R)
@pytest.mark.parametrize("n", [1, 2, 100, 300, 1001, 5000])
def test_rod(n, r):
    u0, gl, gr = _data(n, n)
    u = torch.from_numpy(u0.copy()).cuda()
    ge.Plan(n, r, "fp32", g_left=gl, g_right=gr).step_n(u, 0, 60)
    np.testing.assert_array_equal(u.cpu().numpy(), _rod(u0, r, 60, gl, gr))


@pytest.mark.parametrize("r", [0.5, 1.37])
@pytest.mark.parametrize("n", [99, 700, 5000])
def test_rod_with_a_source(n, r):
    u0, gl, gr = _data(n, n)
    h = 1.0 / (n + 1)
    a = np.linspace(1.0, 0.5, 60)
    b = (3000.0 * np.linspace(0.1, 1.0, n)).astype(F)
    u = torch.from_numpy(u0.copy()).cuda()
    ge.Plan(n, r, "fp32", g_left=gl, g_right=gr, src_b=torch.from_numpy(b).cuda()).step_n(
        u, 0, 60, src_a_t=torch.from_numpy(a).cuda())
    want, tau = u0, r * h * h
    for m in range(60):
        want = _level(want, r, m & 1, gl, gr, (a[m], b, tau))
    np.testing.assert_array_equal(u.cpu().numpy(), want)


@pytest.mark.parametrize("sync", [0, 1, 2, 3])
def test_batch(sync):
    n = np.array([1, 77, 300, 900, 2500, 5000] * len(R), dtype=np.int64)
    offsets = np.zeros(n.size + 1, dtype=np.int64)
    offsets[1:] = np.cumsum((n + 3) // 4 * 4)
    r = np.repeat(R, 6)
    rods = [_data(int(m), i) for i, m in enumerate(n)]
    u0 = np.zeros(int(offsets[-1]), dtype=F)
    for o, (v, _, _) in zip(offsets, rods):
        u0[o:o + v.size] = v
    batch = ge.Batch(n, offsets, r, [g for _, g, _ in rods], [g for _, _, g in rods], "fp32",
                     sync=sync)
    u = torch.from_numpy(u0).cuda()
    batch.solve(u, 0, 40, batch.new_workspace())
    got = u.cpu().numpy()
    for i, (v, gl, gr) in enumerate(rods):
        np.testing.assert_array_equal(got[offsets[i]:offsets[i] + v.size],
                                      _rod(v, r[i], 40, gl, gr), err_msg=str((n[i], r[i])))


@pytest.mark.parametrize("rx,ry", [(0.5, 1.0), (1.0, 0.25), (1.37, 2.0)])
@pytest.mark.parametrize("nx,ny", [(37, 41), (131, 70)])
def test_grid(nx, ny, rx, ry):
    rng = np.random.default_rng(nx)
    u0 = (np.outer(np.sin(np.pi * np.arange(1, ny + 1) / (ny + 1)),
                   np.sin(np.pi * np.arange(1, nx + 1) / (nx + 1))) +
          0.05 * rng.standard_normal((ny, nx))).astype(F)
    walls = (0.25, -0.5, 0.125, 0.75)
    u = torch.from_numpy(u0.copy()).cuda()
    ge.step2d_n(u, nx, ny, rx, ry, 0, 30, "fp32", walls)
    want = u0
    for m in range(30):
        want = _level(want, rx, m & 1, walls[0], walls[1], grid=True).T
        want = _level(want, ry, m & 1, walls[2], walls[3], grid=True).T
    np.testing.assert_array_equal(u.cpu().numpy(), want)
