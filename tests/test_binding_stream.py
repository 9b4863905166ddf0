"""The stream handle the binding passes: the given stream's, or the current
stream's, also with a torch that lacks the private names it reads it through."""

import types

import pytest

torch = pytest.importorskip("torch")

from paper_1808_10481_amd import hl  # noqa: E402


def test_given_stream():
    assert hl._stream_ptr(types.SimpleNamespace(cuda_stream=77)) == 77


@pytest.mark.parametrize("names", [("_cuda_getCurrentRawStream",), ("_cuda_getDevice",)])
def test_current_stream_through_the_public_call(monkeypatch, names):
    for name in names:
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    if names == ("_cuda_getCurrentRawStream",):
        monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    assert hl._stream_ptr(None) == 1234
