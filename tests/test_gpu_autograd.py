"""GPU: the ELBO as a torch.autograd.Function (forward = ELBO kernel, backward = adjoint
kernel with pixel terms recomputed) against central differences and the oracle gradient."""
import sys

import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1803_00113_amd import api, autograd  # noqa: E402
from synth import gen  # noqa: E402


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def test_gradcheck_fp64_path():
    """torch.autograd.gradcheck (central differences in float64) on the float64 pixel path."""
    say("case: gradcheck fp64")
    prob = gen.crop_patches(gen.subset(gen.config2(n_sources=3), images=[2, 4]), 12)
    ctx = api.Context(0, pixel_fp64=True)
    plan = api.Plan(ctx, prob)
    th = torch.as_tensor(prob.theta0, device="cuda").clone().requires_grad_(True)
    f = lambda t: autograd.elbo(plan, t)
    assert torch.autograd.gradcheck(f, (th,), eps=1e-6, atol=1e-5, rtol=1e-6, nondet_tol=0.0)


def test_value_and_gradient_modes():
    """With and without a gradient wanted: the same value; the backward's gradient is the
    library's at the forward's theta, once and repeated; theta changed in place is refused."""
    say("case: autograd value and gradient modes")
    prob = gen.crop_patches(gen.subset(gen.config2(n_sources=3), images=[2, 4]), 12)
    plan = api.Plan(api.Context(0), prob)
    th = torch.as_tensor(prob.theta0, device="cuda").clone().requires_grad_(True)
    tot, _, g = api.elbo_grad(plan, th.detach())
    with torch.no_grad():
        v0 = autograd.elbo(plan, th)
    v1, v2 = autograd.elbo(plan, th), autograd.ElboFunction.apply(th, plan)
    assert not v0.requires_grad and not autograd.elbo(plan, th.detach()).requires_grad
    assert v0.item() == v1.item() == v2.item() == tot.item()
    (3.0 * v1).backward(retain_graph=True)
    assert torch.equal(th.grad, 3.0 * g)
    v1.backward()
    v2.backward()
    assert torch.equal(th.grad, 3.0 * g + g + g)
    v3 = autograd.elbo(plan, th)
    with torch.no_grad():
        th.add_(1e-3)
    with pytest.raises(RuntimeError):
        v3.backward()
