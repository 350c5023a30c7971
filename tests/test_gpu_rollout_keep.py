"""Rollout gradients with the last segment kept from the forward pass against
the same with every segment recomputed: the same kernels on the same inputs,
so equal bit for bit, also on a second backward (which recomputes) and where
segments before the last one follow."""
import pytest
import torch

import paper_2408_02350_amd.adjoint as A
from paper_2408_02350_amd.inputs import CavityConfig

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def problem(kind, dim, precision):
    cav = CavityConfig("keep", dim, 9 if dim == 2 else 6, 8, 4.0, 2.4, 0.8, 0.1, 1, 0)
    if kind == "moving":
        return A.MovingCavity(cav, device=DEV, seed=1, precision=precision)
    return A.FrozenCavity(cav, device=DEV, seed=1, precision=precision,
                          keep_states=kind == "kept")


def inputs(p, kind):
    f0 = p.rest_state().mul_(1.01).requires_grad_(True)
    lid = torch.tensor(0.1, dtype=torch.float64, device=DEV, requires_grad=True)
    return [f0, lid] + ([p.x0.clone().requires_grad_(True)] if kind == "moving" else [])


def rollout(p, kind, ins, nsteps, every):
    if kind == "moving":
        return A.rollout_objective_move(p, ins[0], ins[1], nsteps, every, x0=ins[2])
    return A.rollout_objective(p, ins[0], ins[1], nsteps, every)


@pytest.mark.parametrize("kind", ["kept", "states", "moving"])
@pytest.mark.parametrize("dim,precision,nsteps,every", [
    (2, "fp64", 0, 3), (2, "fp64", 1, 3), (2, "fp32", 3, 3), (2, "fp64", 5, 2), (3, "fp64", 4, 2),
])
def test_kept_last_segment_changes_no_bit(monkeypatch, kind, dim, precision, nsteps, every):
    p = problem(kind, dim, precision)
    ins = inputs(p, kind)
    J = rollout(p, kind, ins, nsteps, every)
    got = [torch.autograd.grad(J, ins, retain_graph=True) for _ in range(2)]
    # two graphs at a time, backward in the order they were built
    Js = [rollout(p, kind, ins, nsteps, every) for _ in range(2)]
    got += [torch.autograd.grad(j, ins) for j in Js]
    monkeypatch.setattr(A, "_room", lambda nbytes, device: False)
    Jr = rollout(p, kind, ins, nsteps, every)
    want = torch.autograd.grad(Jr, ins)
    assert all(torch.equal(j, Jr) for j in [J] + Js)
    for g in got:
        assert all(torch.equal(a, b) for a, b in zip(g, want))
    with torch.no_grad():
        assert torch.equal(rollout(p, kind, ins, nsteps, every), Jr)


def test_an_input_changed_before_the_backward_is_refused():
    p = problem("kept", 2, "fp64")
    ins = inputs(p, "kept")
    J = rollout(p, "kept", ins, 2, 2)
    with torch.no_grad():
        ins[0].mul_(1.5)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        J.backward()
