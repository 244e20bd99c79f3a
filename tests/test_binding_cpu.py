"""The Python binding's own choices, on the CPU."""
import types

import pytest

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def binding():
    import paper_2311_16121_amd._lib as binding
    return binding


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_stream_handle_without_torchs_private_calls(binding, monkeypatch, missing):
    """A torch without one of the private calls gives its current stream's
    handle through the public one."""
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 1000 + d, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert binding._stream(None).value == 1003
    assert binding._stream(types.SimpleNamespace(cuda_stream=55)).value == 55
    monkeypatch.delattr(torch._C, missing)
    assert binding._stream(None).value == 77


def test_outputs_are_plain_tensors(binding):
    """Queries of a tensor subclass decode into an ordinary tensor."""
    class Queries(torch.Tensor):
        pass

    mat = types.SimpleNamespace(out_dim=5)
    for q in (torch.zeros(3, 3), torch.zeros(3, 3).as_subclass(Queries), torch.nn.Parameter(torch.zeros(3, 3))):
        out = binding._out(mat, q, None)
        assert type(out) is torch.Tensor and out.shape == (3, 5) and out.dtype == torch.float32
        assert not out.requires_grad
