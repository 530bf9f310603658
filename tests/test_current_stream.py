"""The stream of a call without a given one: torch's current stream, by its
private calls where a torch has them and by the public one where not."""
import types

import pytest

import paper_2604_21117_amd as g


@pytest.mark.parametrize("private", [(), ("_cuda_getDevice",), ("_cuda_getDevice", "_cuda_getCurrentRawStream")])
def test_current_stream(monkeypatch, private):
    now = {"device": 1, 0: 100, 1: 101}
    calls = {"_cuda_getDevice": lambda: now["device"], "_cuda_getCurrentRawStream": lambda d: now[d]}
    cuda = types.SimpleNamespace(current_stream=lambda: types.SimpleNamespace(cuda_stream=now[now["device"]]))
    fake = types.SimpleNamespace(cuda=cuda, _C=types.SimpleNamespace(**{f: calls[f] for f in private}))
    monkeypatch.setattr(g, "_torch", lambda: fake)
    monkeypatch.setattr(g, "_raw_stream", None)
    assert [g._stream(None), g._stream(None)] == [101, 101]
    now[1] = 111
    assert g._stream(None) == 111
    now["device"] = 0
    assert g._stream(None) == 100
    assert g._stream(types.SimpleNamespace(cuda_stream=7)) == 7
