"""The layers' products at the edges of how they are split over workgroups."""
import numpy as np
import pytest

from oracle import conv_ref as cr
from paper_1310_3422_amd import ge

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# one FP32 addition errs by at most 2^-24 of its result; 2^-23 leaves room for
# a matrix core that truncates
ACC_U = 2.0 ** -23


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to(torch.bfloat16).cuda()


def _close(got, want, mag, k):
    err = np.abs(got - want) - (k - 1) * ACC_U * mag
    assert np.all(err <= 1e-300), float(err.max())


# segments of 128 positions: one, an odd number, a rod of one segment each,
# and more pairs of them than there are workgroups
@pytest.mark.parametrize("layer", [1, 3, 5, 6])
@pytest.mark.parametrize("batch,width", [(1, 128), (3, 128), (1, 384), (5, 640), (131, 512)])
def test_products_at_the_edges_of_the_split(layer, batch, width):
    rng = np.random.default_rng([layer, batch, width])
    net = ge.Net(width=width, max_batch=batch, seed=1)
    ci, co, cip, cop, cod, dil = ge.Net.layer_shape(layer)
    flat, at = net.params(), sum(5 * a * b + b for a, b in cr.LAYERS[:layer - 1])
    w = cr.bf16(flat[at:at + 5 * co * ci].reshape(5, co, ci).astype(np.float64))
    x = np.zeros((batch, width, cip))
    x[:, :, :ci] = cr.bf16(rng.standard_normal((batch, width, ci)))
    g = np.zeros((batch, width, cod))
    g[:, :, :co] = cr.bf16(rng.standard_normal((batch, width, co)))
    xd, gd, xr, gr = _dev(x), _dev(g), x[:, :, :ci], g[:, :, :co]
    some = np.unique(np.linspace(0, batch - 1, min(batch, 6)).astype(int))   # rods compared
    fwd = net.layer_probe(layer, 0, batch, x=xd).cpu().numpy()[some, :, :co].astype(np.float64)
    _close(fwd, cr.conv(xr[some], w, dil), cr.conv(np.abs(xr[some]), np.abs(w), dil), 5 * ci + 1)
    if layer > 1:
        dx = net.layer_probe(layer, 1, batch, g=gd).cpu().numpy()[some, :, :ci].astype(np.float64)
        _close(dx, cr.conv_input_grad(gr[some], w, dil),
               cr.conv_input_grad(np.abs(gr[some]), np.abs(w), dil), 5 * co)
    out = net.layer_probe(layer, 2, batch, x=xd, g=gd).cpu().numpy().astype(np.float64)
    xp, npos = np.pad(xr, ((0, 0), (2 * dil, 2 * dil), (0, 0))), batch * width
    for k in range(5):
        xk = xp[:, k * dil:k * dil + width].reshape(npos, ci)
        gk = gr.reshape(npos, co)
        _close(out[k * co * ci:(k + 1) * co * ci].reshape(co, ci), gk.T @ xk,
               np.abs(gk).T @ np.abs(xk), npos)
    _close(out[5 * co * ci:], gr.sum(axis=(0, 1)), np.abs(gr).sum(axis=(0, 1)), npos)
