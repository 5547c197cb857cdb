"""Which evaluations the ELBO's autograd function makes (the library's calls replaced by host
functions that count): one for a value and its gradient through elbo(); a value alone where
no gradient can be wanted, and by ElboFunction.apply, whose gradient waits for a backward."""
import pytest

torch = pytest.importorskip("torch")

from paper_1803_00113_amd import autograd  # noqa: E402


@pytest.fixture
def calls(monkeypatch):
    made = []

    def value(plan, th):
        assert not th.requires_grad
        return (th ** 3).sum().reshape(1), None

    def elbo_eval(plan, th):
        made.append("value")
        return value(plan, th)

    def elbo_grad(plan, th):
        made.append("gradient")
        return (*value(plan, th), 3 * th.double() ** 2)

    monkeypatch.setattr(autograd.api, "elbo_eval", elbo_eval)
    monkeypatch.setattr(autograd.api, "elbo_grad", elbo_grad)
    return made


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_evaluations(calls, dtype):
    th = torch.linspace(-1, 2, 8, dtype=dtype).reshape(2, 4).requires_grad_(True)
    want = 3 * th.detach() ** 2

    def grad_of(v):
        th.grad = None
        v.backward(retain_graph=True)
        assert th.grad.dtype == dtype and torch.allclose(th.grad, want)

    v = autograd.elbo("plan", th)
    grad_of(v)
    grad_of(v)
    assert calls == ["gradient"]
    del calls[:]
    with torch.no_grad():
        assert autograd.elbo("plan", th).item() == v.item()
        assert not autograd.ElboFunction.apply(th, "plan").requires_grad
    assert autograd.elbo("plan", th.detach()).item() == v.item()
    assert calls == ["value"] * 3
    del calls[:]
    v = autograd.ElboFunction.apply(th, "plan")
    assert calls == ["value"]
    grad_of(v)
    assert calls == ["value", "gradient"]
    v = autograd.ElboFunction.apply(th, "plan")
    with torch.no_grad():
        th.add_(1.0)
    with pytest.raises(RuntimeError):
        v.backward()
