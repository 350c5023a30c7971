"""What a rollout holds between its two passes, on the CPU: the library calls
are stand-ins that read and write through the tensors' storage, as the library
does, so that no tensor's version tells of a write."""
import types

import pytest
import torch

import paper_2408_02350_amd.adjoint as A

F64 = torch.float64


def put(dst, src):
    dst.detach().numpy()[...] = src.detach().numpy()  # the version of dst stays


class Kernels:
    """A step f' = c f + a U f^2 + lid, U' = mean f, and its adjoint, exact."""
    c, a = 0.9, 0.05

    def __init__(self):
        self.lid, self.calls = 0.0, []

    def bgk_set_lid_velocity(self, ctx, lid):
        self.lid = lid

    def bgk_moments(self, ctx, f):
        return f.new_ones(1), f.detach().mean().reshape(1, 1), f.new_ones(1)

    def bgk_step(self, ctx, f, fn, x, U, rho, T):
        self.calls.append("step")
        out = self.c * f + self.a * U * f * f + self.lid + 0.01 * x.sum()
        put(fn, out)
        put(U, out.mean().reshape(1, 1))
        if ctx.moves:
            put(x, x * 1.01)

    def bgk_step_keep(self, ctx, f, fn, x, U, rho, T, ft):
        self.bgk_step(ctx, f, fn, x, U, rho, T)
        put(ft, f)

    def bgk_objective(self, ctx, f, rho, U, ke, want_grad):
        J = (f * f).sum()
        return (J, (2 * f, torch.zeros_like(rho), torch.zeros_like(U))) if want_grad else J

    def bgk_adjoint_step(self, ctx, f, U, x, l1, lU1, lr, lT, lf, lU, dlid):
        g = l1 + lU1 / f.numel()
        put(dlid, dlid + g.sum())
        put(lU, (g * self.a * f * f).sum().reshape(1, 1))
        put(lf, g * (self.c + 2 * self.a * U * f))

    def bgk_adjoint_step_kept(self, ctx, f, U, x, kept, *rest):
        assert torch.equal(kept[0], f)
        self.bgk_adjoint_step(ctx, f, U, x, *rest)

    def bgk_adjoint_step_move(self, ctx, f, U, x, l1, lU1, lx1, lr, lT, lf, lU, lx, dlid):
        g = (l1 + lU1 / f.numel()).sum()
        put(lx, 1.01 * lx1 + 0.01 * g)
        self.bgk_adjoint_step(ctx, f, U, x, l1, lU1, lr, lT, lf, lU, dlid)

    def bgk_moments_adjoint(self, ctx, rho, U, T, lf, lr, lU, lT):
        put(lf, lf + lU / lf.numel())


@pytest.fixture
def kernels(monkeypatch):
    k = Kernels()
    monkeypatch.setattr(A, "B", k)
    monkeypatch.setattr(A, "_room", lambda nbytes, device: True)
    return k


def problem(kind):
    base = A.MovingCavity if kind == "moving" else A.FrozenCavity
    p = object.__new__(base)
    p.ctx = types.SimpleNamespace(device="cpu", moves=kind == "moving")
    p.N = 1
    if kind != "moving":  # (a moving cavity without the attribute keeps states)
        p.keep_states = kind != "states"
    p.x = p.x0 = torch.full((1, 1), 0.5, dtype=F64)
    return p


def inputs():
    f0 = torch.linspace(0.5, 1.5, 6, dtype=F64).requires_grad_(True)
    return f0, torch.tensor(0.1, dtype=F64, requires_grad=True)


def rollout(p, f0, lid, nsteps, every):
    call = A.rollout_objective_move if isinstance(p, A.MovingCavity) else A.rollout_objective
    return call(p, f0, lid, nsteps, every)


KINDS = ["kept", "states", "moving"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("nsteps,every", [(3, 3), (5, 2)])
def test_a_write_into_f0_before_the_backward_does_not_reach_the_steps(kernels, kind, nsteps, every):
    # (the moments of f^0, which enter its own gradient alone, are the caller's)
    p = problem(kind)
    f0, lid = inputs()
    want, = torch.autograd.grad(rollout(p, f0, lid, nsteps, every), lid)
    J = rollout(p, f0, lid, nsteps, every)
    put(f0, 3 * f0)
    for _ in range(2):
        assert torch.equal(torch.autograd.grad(J, lid, retain_graph=True)[0], want)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("nsteps,every", [(3, 3), (5, 2)])
def test_copying_hooks_hold_f0_as_it_was(kernels, kind, nsteps, every):
    p = problem(kind)
    f0, lid = inputs()
    want = torch.autograd.grad(rollout(p, f0, lid, nsteps, every), [f0, lid])
    with torch.autograd.graph.saved_tensors_hooks(torch.clone, lambda t: t):
        J = rollout(p, f0, lid, nsteps, every)
    with torch.no_grad():
        f0.mul_(3)
    for _ in range(2):
        got = torch.autograd.grad(J, [f0, lid], retain_graph=True)
        assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("where", ["class", "instance"])
def test_a_problem_with_its_own_forward_is_asked_for_the_whole_rollout(kernels, kind, where):
    p = problem(kind)
    own, seen = type(p).forward, []

    def forward(self, f0, lid, nsteps, every=None, *more):
        seen.append((nsteps, every))
        return own(self, f0, lid, nsteps, every, *more)

    f0, lid = inputs()
    want = torch.autograd.grad(rollout(p, f0, lid, 3, 2), [f0, lid])
    if where == "class":
        p.__class__ = type("Own", (type(p),), {"forward": forward})
    else:
        p.forward = types.MethodType(forward, p)
    got = torch.autograd.grad(rollout(p, f0, lid, 3, 2), [f0, lid])
    assert seen == [(3, 2)]
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("kind", ["frozen", "moving"])
@pytest.mark.parametrize("nsteps,every", [(3, 3), (5, 2)])
def test_without_keep_states_only_segment_starts_wait_for_the_backward(kernels, kind, nsteps,
                                                                       every):
    p = problem(kind)
    f0, lid = inputs()
    want = torch.autograd.grad(rollout(p, f0, lid, nsteps, every), [f0, lid])
    p.keep_states = False
    kernels.calls.clear()
    J = rollout(p, f0, lid, nsteps, every)
    assert J.grad_fn.last is None and sorted(J.grad_fn.saved) == list(range(0, nsteps, every))
    assert len(kernels.calls) == nsteps
    got = torch.autograd.grad(J, [f0, lid])
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("free,reserved,allocated,room", [
    (400, 0, 0, True), (399, 0, 0, False), (0, 900, 500, True), (0, 900, 501, False),
    (300, 200, 100, True),
])
def test_room_counts_what_the_allocator_holds_unused(monkeypatch, free, reserved, allocated, room):
    cuda = {"is_current_stream_capturing": lambda: False, "mem_get_info": lambda d: (free, 1000),
            "memory_reserved": lambda d: reserved, "memory_allocated": lambda d: allocated}
    for name, fn in cuda.items():
        monkeypatch.setattr(torch.cuda, name, fn)
    assert A._room(100, "cuda:0") is room


@pytest.mark.parametrize("kind", ["kept", "moving"])
@pytest.mark.parametrize("nsteps,every", [(3, 3), (5, 2)])
def test_the_kept_segment_is_not_run_again_but_by_a_second_backward(kernels, kind, nsteps, every):
    p = problem(kind)
    f0, lid = inputs()
    J = rollout(p, f0, lid, nsteps, every)
    assert J.grad_fn.last is not None and len(kernels.calls) == nsteps
    ran = []
    for _ in range(2):
        kernels.calls.clear()
        torch.autograd.grad(J, [f0, lid], retain_graph=True)
        ran.append(len(kernels.calls))
    # a segment of n steps: n run with all that the reverse reads, or its n states in n - 1
    run = [b - a - (kind == "moving") for a, b in A.segments(nsteps, every)]
    assert ran == [sum(run[:-1]), sum(run)]


@pytest.mark.parametrize("kind", ["kept", "moving"])
def test_graphs_side_by_side_keep_a_quarter_together(monkeypatch, kernels, kind):
    monkeypatch.undo()
    monkeypatch.setattr(A, "B", kernels)
    p = problem(kind)
    f0, lid = inputs()
    segment = 3 * (2 if kind == "kept" else 1) * f0.numel() * f0.element_size()
    total = 9 * segment  # room for two segments, not for a third

    def kept():
        return sum(len(k) * k.step_bytes for k in A._live)

    cuda = {"is_current_stream_capturing": lambda: False, "memory_reserved": lambda d: 0,
            "mem_get_info": lambda d: (total - kept(), total), "memory_allocated": lambda d: 0}
    for name, fn in cuda.items():
        monkeypatch.setattr(torch.cuda, name, fn)
    Js = [rollout(p, f0, lid, 3, 3) for _ in range(4)]
    assert [J.grad_fn.last is not None for J in Js] == [True, True, False, False]
    assert kept() == 2 * segment
    torch.autograd.grad(Js[0], lid)  # used up
    Js[1] = None                     # dropped
    assert kept() == 0
    assert rollout(p, f0, lid, 3, 3).grad_fn.last is not None
