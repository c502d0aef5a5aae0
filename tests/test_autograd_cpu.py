"""The differentiable objective's rule around its two evaluations, on the CPU:
the evaluation is replaced by one that writes given scalars and gradients."""
import pytest
import torch

from paper_1312_4587_amd import autograd, fftpl

LAM = 0.75


class _Prob:
    fast = True


@pytest.fixture
def objective(monkeypatch):
    gen = torch.Generator().manual_seed(7)
    x, y, dx, dy = (torch.rand(37, generator=gen) for _ in range(4))

    def eval_(plan, prob, x_, y_, lam, gamma, mode, gx, gy, out4):
        assert mode == "exact" and (gx is None) == (gy is None)
        out4.copy_(torch.tensor([3.0, 5.0, 7.0, 0.5], dtype=torch.float64))
        if gx is not None:
            gx.copy_(dx)
            gy.copy_(dy)

    monkeypatch.setattr(fftpl, "eval", eval_)

    def call():
        x.grad = y.grad = None
        x.requires_grad_(True)
        y.requires_grad_(True)
        loss, scalars = autograd.objective(x, y, None, _Prob(), LAM, 1.0)
        return x, y, loss, scalars

    return call, dx, dy


def test_gradient_is_scaled_in_float32(objective):
    call, dx, dy = objective
    x, y, loss, scalars = call()
    assert loss.dtype == torch.float64 and loss.item() == 5.0 + LAM * 3.0
    assert not scalars.requires_grad
    (loss / 3.0).backward()
    s = torch.tensor(1.0 / 3.0, dtype=torch.float64).to(torch.float32)
    assert x.grad.dtype == torch.float32
    assert torch.equal(x.grad, dx * s) and torch.equal(y.grad, dy * s)


# several incoming gradients at once: torch runs the backward once under vmap
def test_batched_incoming_gradients(objective):
    call, dx, dy = objective
    x, y, loss, _ = call()
    g = torch.tensor([1.0, -2.5, 1.0 / 3.0], dtype=torch.float64)
    gx, gy = torch.autograd.grad(loss, (x, y), g, is_grads_batched=True)
    assert gx.dtype == torch.float32 and gx.shape == (3, 37)
    for k in range(3):
        s = g[k].to(torch.float32)
        assert torch.equal(gx[k], dx * s) and torch.equal(gy[k], dy * s)


# an incoming gradient that itself needs a gradient
def test_backward_is_differentiable_in_the_incoming_gradient(objective):
    call, dx, dy = objective
    x, y, loss, _ = call()
    s = torch.tensor(2.0, dtype=torch.float64, requires_grad=True)
    gx, gy = torch.autograd.grad(loss, (x, y), s, create_graph=True)
    (ds,) = torch.autograd.grad(gx.sum() + gy.sum(), s)
    assert abs(ds.item() - (dx.sum() + dy.sum()).item()) < 1e-4
