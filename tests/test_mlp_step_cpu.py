"""The training step's bookkeeping and its route, without a GPU: a batch that is refused
leaves the step count alone (it enters Adam's bias correction), and a subclass's own
forward and backward are called."""
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
