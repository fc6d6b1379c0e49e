"""The objective's backward where gradients of several outputs are asked for at once: torch runs it under vmap then, on a
batched output gradient. The library's calls are replaced by fixed tensors, so this needs no GPU."""
import pytest

torch = pytest.importorskip("torch")


@pytest.fixture
def objective(monkeypatch):
    import paper_2412_14973_amd as tl
    gen = torch.Generator().manual_seed(1)
    g = torch.complex(torch.randn(7, generator=gen), torch.randn(7, generator=gen))
    monkeypatch.setattr(tl, "forward", lambda *a, **k: (torch.tensor(2.5, dtype=torch.float64), None, None))
    monkeypatch.setattr(tl, "grad", lambda *a, **k: (None, g.clone()))
    return lambda theta: tl.objective(theta, None, None, None), g


def test_backward(objective):
    f, g = objective
    theta = torch.zeros(7, dtype=torch.complex64, requires_grad=True)
    (3.0 * f(theta)).backward()
    assert theta.grad.dtype == torch.complex64 and torch.equal(theta.grad, 3.0 * g)


def test_batched_output_gradients(objective):
    f, g = objective
    theta = torch.zeros(7, dtype=torch.complex64, requires_grad=True)
    weights = torch.tensor([1.0, -2.0, 0.5], dtype=torch.float64)
    (got,) = torch.autograd.grad(f(theta), theta, weights, is_grads_batched=True)
    assert got.dtype == torch.complex64
    assert torch.equal(got, weights.to(torch.float32)[:, None] * g)


def test_output_gradient_stays_in_the_graph(objective):
    f, g = objective
    theta = torch.zeros(7, dtype=torch.complex64, requires_grad=True)
    scale = torch.tensor(1.5, dtype=torch.float64, requires_grad=True)
    (got,) = torch.autograd.grad(scale * f(theta), theta, create_graph=True)
    (ds,) = torch.autograd.grad(got.abs().square().sum(), scale)
    assert torch.allclose(ds, 2 * 1.5 * g.abs().square().sum().double(), rtol=1e-5)
