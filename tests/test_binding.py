"""The Python binding without a GPU: it imports on a torch that lacks the
undocumented stream calls, and makes its fp32 outputs fp32 whatever buffers the
caller passes beside them."""
import importlib.util
import types

import pytest
import torch

from paper_2402_17152_amd import hstu


@pytest.mark.parametrize("name", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_imports_and_finds_the_stream_without_private_calls(monkeypatch, name):
    monkeypatch.delattr(torch._C, name, raising=False)
    spec = importlib.util.spec_from_file_location("hstu_copy", hstu.__file__)
    mod = importlib.util.module_from_spec(spec)
    mod.__package__ = hstu.__package__
    spec.loader.exec_module(mod)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda: types.SimpleNamespace(cuda_stream=1234))
    assert mod._stream() == 1234
    assert mod._stream(types.SimpleNamespace(cuda_stream=7)) == 7


def test_layer_statistics_are_fp32_beside_a_callers_buffer(monkeypatch):
    T, H, d = 5, 2, 32
    q = torch.zeros(T, H, d, dtype=torch.bfloat16)
    u = torch.zeros(T, H * d, dtype=torch.bfloat16)
    offs = torch.tensor([0, T])
    ts = torch.zeros(T, dtype=torch.int64)
    tab = torch.zeros(2 * T - 1)
    calls = types.SimpleNamespace(hstu_layer_fwd=lambda *a: 0)
    monkeypatch.setattr(hstu, "lib", calls)
    for dtype in (torch.float32, torch.int32, torch.float64):
        buf = torch.zeros(T, H * d, dtype=dtype)  # room for T * H * d floats
        out, y, mean, rstd = hstu.hstu_layer_fwd(
            q, q, q, u, offs, ts, tab, torch.zeros(4), T, attn_out=buf,
            ws=torch.zeros(256, dtype=torch.uint8), stream=types.SimpleNamespace(cuda_stream=0))
        assert out is buf and y.dtype == torch.bfloat16
        assert mean.dtype == rstd.dtype == torch.float32
