"""The stream handle of a call on device tensors, with torch's device functions
replaced (no device)."""
import types

import numpy as np
import pytest
import torch

from paper_1309_2710_amd import rkc


def test_autotune_refuses_cpu_tensors(monkeypatch):
    """Host memory is never handed on as device arrays."""
    calls = []
    rkc.make_opts()   # the library's own defaults, kept from here on
    fake = types.SimpleNamespace(rkc_autotune=lambda *a: calls.append(a) or rkc.OK)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 0)
    monkeypatch.setattr(rkc, "lib", lambda: fake)
    mech = types.SimpleNamespace(handle=None, n_species=2)
    T, P, Y = (torch.from_numpy(np.ones(s)) for s in ((3,), (3,), (3, 2)))
    with pytest.raises(ValueError):
        rkc.autotune(mech, T, P, Y, 1e-6)
    assert not calls


def test_public_stream_where_the_raw_handle_is_missing(monkeypatch):
    """The raw handle is a private name of torch: without it, the public call."""
    t = types.SimpleNamespace(get_device=lambda: 3)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 1000 + d)
    assert rkc._stream_handle(None, [t]).value == 1003
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda d: types.SimpleNamespace(cuda_stream=2000 + d))
    assert rkc._stream_handle(None, [t]).value == 2003
