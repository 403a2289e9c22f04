"""The training step's bookkeeping, route and argument checks, without a GPU: a batch that
is refused leaves the step count alone (it enters Adam's bias correction), a subclass's own
forward and backward are called, and every shape and type the kernels rely on is
checked before the call."""
import ctypes
import os

import pytest
import torch

from paper_2410_04477_amd import api
from paper_2410_04477_amd.warmstart import MLP


@pytest.mark.parametrize("batch", [0, 8])
def test_refused_batch_does_not_count(batch):
    net = MLP(1, "cpu")
    with pytest.raises(Exception):
        net.train_step(torch.zeros(batch, 96), torch.zeros(batch, 3), 1e-3)   # not on the HIP device
    assert net.step_count == 0


def test_overridden_methods_are_called(monkeypatch):
    calls = []

    class Sub(MLP):
        def forward(self, X):
            calls.append("forward")
            return torch.zeros(X.shape[0], 3), None

        def backward(self, cache, dout):
            calls.append("backward")
            return [torch.zeros_like(p) for p in self.params]

    monkeypatch.setattr(api, "mse", lambda out, T, dout: torch.zeros(8))
    monkeypatch.setattr(api, "adam", lambda *a, **k: calls.append("adam"))
    monkeypatch.setattr(api, "mlp_step", lambda *a, **k: pytest.fail("the one-call step ignores the subclass"))
    net = Sub(1, "cpu")
    net.train_step(torch.zeros(4, 96), torch.zeros(4, 3), 1e-3)
    assert calls == ["forward", "backward"] + ["adam"] * 6 and net.step_count == 1


def _case(**change):
    z = lambda *s, dt=torch.float32: torch.zeros(*s, dtype=dt)
    shapes = [(16, 12), (16,), (16, 16), (16,), (3, 16), (3,)]
    kw = dict(X=z(5, 12), target=z(5, 3), sizes=(12, 16, 16, 3), params=[z(*s) for s in shapes],
              m=[z(*s) for s in shapes], v=[z(*s) for s in shapes], step=1)
    kw.update(change)
    return kw


Z = torch.zeros


@pytest.mark.parametrize("change", [
    dict(X=Z(5, 11)), dict(X=Z(60)), dict(X=Z(5, 12, dtype=torch.float64)), dict(target=Z(4, 3)), dict(target=Z(5, 2)),
    dict(target=Z(5, 3, dtype=torch.float16)), dict(sizes=(12, 16, 3)), dict(params=_case()["params"][:5]),
    dict(m=_case()["m"][:4] + [Z(3, 15), Z(3)]), dict(v=[Z(16, 12, dtype=torch.float64)] + _case()["v"][1:])])
def test_shapes_and_types_are_checked(change):
    with pytest.raises(ValueError, match="sizes|float32|batch|values per row|weight"):
        api.mlp_step(**_case(**change))


def test_well_formed_arguments_reach_the_device_check():
    with pytest.raises(ValueError, match="HIP device"):
        api.mlp_step(**_case())


@pytest.mark.skipif(not os.path.exists(os.path.join(os.path.dirname(api.__file__), "libvecchia.so")), reason="library not built")
@pytest.mark.parametrize("batch,width,ok", [(256, 3, True), (1 << 20, 2031, True), (1 << 20, 2047, False),
                                            (1 << 20, 16384, False), (65536, 16384, True), (131072, 16384, False)])
def test_outputs_are_counted_in_32_bits(batch, width, ok):
    """More outputs than the loss kernel counts (2^31, less the strides of its grid) have no workspace size."""
    from paper_2410_04477_amd import _lib as L
    size = L.lib().vecchia_mlp_step_workspace_size(batch, (ctypes.c_int32 * 4)(16, 16, 16, width))
    assert (size > 0) == ok
