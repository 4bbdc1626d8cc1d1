"""Host-side argument checks of the FP4 Linear layer (no GPU: the layer is
built on the CPU; where it runs, the library calls are replaced)."""

import pytest
import torch

from paper_2609_02846_amd import linear
from paper_2609_02846_amd.linear import Linear


def test_block_size_and_shape_checks():
    assert Linear(64, 96, device="cpu", block=32).block == 32
    assert Linear(48, 80, device="cpu").block == 16
    with pytest.raises(ValueError):
        Linear(48, 64, device="cpu", block=32)            # 48 is not a multiple of 32
    with pytest.raises(ValueError):
        Linear(64, 64, device="cpu", block=8)
    with pytest.raises(ValueError):
        Linear(64, 64, device="cpu", block=32, rht_wgrad=True)
    with pytest.raises(ValueError):
        Linear(40, 64, device="cpu")
    with pytest.raises(ValueError):
        Linear(64, 64, device="cpu", grad_rounding="stochastic")


class _NoLibrary:
    """Every library call succeeds and does nothing."""

    def __getattr__(self, name):
        return lambda *args: 0


def test_unknown_gradient_rounding_is_refused(monkeypatch):
    """A rounding assigned after construction that is neither "sr" nor "rn"
    must not run as round to nearest."""
    layer = Linear(32, 48, device="cpu")
    monkeypatch.setattr(linear, "load_library", _NoLibrary)
    monkeypatch.setattr(linear, "_stream", lambda: 0)
    for check in ("_bf16_2d", "_f32_out", "_dev_buf"):
        monkeypatch.setattr(linear, check, lambda t, *a: t)
    x = torch.zeros(16, 32, dtype=torch.bfloat16, requires_grad=True)
    for known in ("sr", "rn"):
        layer.grad_rounding = known
        layer(x).sum().backward()
    layer.grad_rounding = "SR"
    y = layer(x)
    with pytest.raises(KeyError):
        y.sum().backward()
