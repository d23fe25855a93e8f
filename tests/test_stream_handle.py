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
