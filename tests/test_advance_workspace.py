"""Net.advance refuses a workspace that is smaller than its batch plan's (the
rods of 4465 points and more need second level buffers), before any call into
the library."""
import types

import pytest

from paper_1310_3422_amd import ge

torch = pytest.importorskip("torch")


def _tensor(numel, size, dtype=None, cuda=True):
    return types.SimpleNamespace(is_cuda=cuda, dtype=dtype, numel=lambda: numel,
                                 element_size=lambda: size, is_contiguous=lambda: True,
                                 data_ptr=lambda: 1 << 20)


@pytest.mark.parametrize("numel,size,cuda,accepted", [
    (256, 1, True, False), (256 + 2 * 8192 * 8 - 1, 1, True, False), (256 + 2 * 8192 * 8, 1, True, True),
    (32 + 2 * 8192, 8, True, True), (1 << 20, 1, False, False)])
def test_workspace_size(monkeypatch, numel, size, cuda, accepted):
    calls = []
    monkeypatch.setattr(ge, "_lib", types.SimpleNamespace(
        ge_nn_advance=lambda *a: calls.append(a) or ge.GE_OK))
    net = ge.Net.__new__(ge.Net)
    net.width, net.handle = 8192, None
    plan = types.SimpleNamespace(handle=None, workspace_bytes=256 + 2 * 8192 * 8)
    u, r = _tensor(2 * 8192, 4, torch.float32), _tensor(2, 4, torch.float32)
    stream = types.SimpleNamespace(cuda_stream=0)
    run = lambda: net.advance(plan, _tensor(numel, size, cuda=cuda), u, r, 4,  # noqa: E731
                              stream=stream)
    if accepted:
        run()
    else:
        with pytest.raises(ValueError, match="ge_ws"):
            run()
    assert len(calls) == accepted
