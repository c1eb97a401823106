"""The default interval between checkpoints of a rollout."""
import pytest
import torch

from paper_1401_0427_amd import adjoint

FACES = ("inflow", "neumann", "wall", "inflow")


@pytest.mark.parametrize("shape,bc,T,K", [
    ((8, 8), ("periodic",) * 4, 80, 8), ((8, 8), ("periodic",) * 4, 500, 24), ((8, 8), ("periodic",) * 4, 30, 5),
    ((8, 8), (0, 0, 0, 0), 80, 8),
    # nothing runs in pairs: sqrt(T) as it is
    ((8, 8), FACES, 80, 9), ((8, 8), ("periodic", "periodic", "wall", "wall"), 500, 22),
    ((8,), ("periodic",) * 4, 80, 9), ((8,), ("neumann", "neumann", "periodic", "periodic"), 500, 22)])
def test_default_interval(monkeypatch, shape, bc, T, K):
    seen = []
    monkeypatch.setattr(adjoint._Rollout, "apply", lambda *a: seen.append(a))
    adjoint.rollout(torch.ones(shape, dtype=torch.float64), torch.tensor(1.8), T, bc=bc)
    adjoint.rollout(torch.ones(shape, dtype=torch.float64), torch.tensor(1.8), T, K=13, bc=bc)
    assert [a[3] for a in seen] == [K, 13]
