"""A rollout whose f^0 the library overwrites between the two passes (no tensor
version tells of it), and one under hooks that copy the saved tensors: the
steps are reversed from f^0 as the forward pass met it, bit for bit."""
import pytest
import torch

import paper_2408_02350_amd.adjoint as A
import paper_2408_02350_amd.bgk as B
from paper_2408_02350_amd.inputs import CavityConfig

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def setup(kind, dim, precision, every):
    cav = CavityConfig("writes", dim, 9 if dim == 2 else 6, 8, 4.0, 2.4, 0.8, 0.1, 1, 0)
    make = A.MovingCavity if kind == "moving" else A.FrozenCavity
    p = make(cav, device=DEV, seed=1, precision=precision)
    f0 = p.rest_state()
    f0.mul_(1.0 + 0.1 * (p.x if kind == "kept" else p.x0)[0].to(f0.dtype)[:, None]).requires_grad_(True)
    lid = torch.tensor(0.1, dtype=torch.float64, device=DEV, requires_grad=True)
    roll = A.rollout_objective_move if kind == "moving" else A.rollout_objective
    return p, f0, lid, lambda: roll(p, f0, lid, 5, every)


@pytest.mark.parametrize("kind", ["kept", "moving"])
@pytest.mark.parametrize("dim,precision", [(2, "fp32"), (3, "fp64")])
def test_a_step_into_f0_before_the_backward(kind, dim, precision):
    p, f0, lid, roll = setup(kind, dim, precision, 2)
    want, = torch.autograd.grad(roll(), lid)
    J = roll()
    x = (p.x if kind == "kept" else p.x0).clone()
    g = p.rest_state().mul_(1.3)
    rho, U, T = B.bgk_moments(p.ctx, g)
    B.bgk_step(p.ctx, g, f0.detach(), x, U, rho, T)
    assert torch.equal(torch.autograd.grad(J, lid)[0], want)


def test_copying_hooks():
    _, f0, lid, roll = setup("kept", 2, "fp64", 5)
    want = torch.autograd.grad(roll(), [f0, lid])
    with torch.autograd.graph.save_on_cpu():
        J = roll()
    with torch.no_grad():
        f0.mul_(1.5)
    for _ in range(2):
        got = torch.autograd.grad(J, [f0, lid], retain_graph=True)
        assert all(torch.equal(a, b) for a, b in zip(got, want))
