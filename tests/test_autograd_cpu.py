"""IQPExpval's backward where a consumer of the mean gives it no gradient: the
gradient of theta is zeros, as with materialised gradients. The library's calls
are replaced by host stand-ins, so no GPU is needed."""
import pytest
import torch

from paper_2501_04776_amd import IQPExpval, api


class _NoGrad(torch.autograd.Function):
    """The sum of x, with no gradient."""

    @staticmethod
    def forward(ctx, x):
        return x.sum()

    @staticmethod
    def backward(ctx, g):
        return None


@pytest.fixture
def host_calls(monkeypatch):
    class Circuit:
        def __init__(self, n, gens, theta):
            self.theta = theta

    def expval(circ, ops, samples, precision, stderr=True, phase_save=False):
        mean = circ.theta.sum() * torch.ones(ops.shape[0], dtype=torch.float64)
        return mean, torch.zeros_like(mean), torch.zeros(ops.shape[0], samples.shape[0])

    def expval_grad(circ, ops, samples, grad_mean, phase_save=None, precision=None):
        assert grad_mean.dtype == torch.float64 and grad_mean.shape == (ops.shape[0],)
        return grad_mean.sum() * torch.ones_like(circ.theta)

    monkeypatch.setattr(api, "Circuit", Circuit)
    monkeypatch.setattr(api, "iqp_expval", expval)
    monkeypatch.setattr(api, "iqp_expval_grad", expval_grad)


def _mean():
    theta = torch.linspace(0.1, 0.5, 5, dtype=torch.float64, requires_grad=True)
    rows = torch.zeros((3, 1), dtype=torch.int64)
    mean, se = IQPExpval.apply(theta, rows, rows, rows, 10, "split_bf16")
    assert not se.requires_grad
    return theta, mean


def test_missing_gradient_of_the_mean_is_zeros(host_calls):
    theta, mean = _mean()
    (g,) = torch.autograd.grad(_NoGrad.apply(mean), theta)
    assert torch.equal(g, torch.zeros_like(theta))
    theta, mean = _mean()
    _NoGrad.apply(mean).backward()
    assert torch.equal(theta.grad, torch.zeros_like(theta))


def test_missing_gradient_beside_another_consumer(host_calls):
    theta, mean = _mean()
    (g,) = torch.autograd.grad(_NoGrad.apply(mean) + 2.0 * mean.sum(), theta)
    assert torch.equal(g, torch.full_like(theta, 6.0))
