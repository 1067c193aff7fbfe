"""The stream a call of the Python binding runs on."""
import types

import pytest

import paper_1908_06091_amd as P


def _torch(raw):
    t = types.SimpleNamespace()
    t.cuda = types.SimpleNamespace(
        current_stream=lambda: types.SimpleNamespace(cuda_stream=77))
    t._C = types.SimpleNamespace()
    if "stream" in raw:
        t._C._cuda_getCurrentRawStream = lambda device: 70 + device
    if "device" in raw:
        t._C._cuda_getDevice = lambda: 5
    return t


@pytest.mark.parametrize("raw,want", [(("stream", "device"), 75), (("stream",), 77),
                                      (("device",), 77), ((), 77)])
def test_current_stream_without_torch_private_calls(monkeypatch, raw, want):
    monkeypatch.setattr(P, "_torch_module", _torch(raw))
    assert P._stream(None) == want


def test_a_given_stream_is_taken():
    assert P._stream(types.SimpleNamespace(cuda_stream=3)) == 3
