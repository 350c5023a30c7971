"""Gradients of a cavity rollout by the hand-written reverse step.

The rollout is the frozen-cloud map (S4-S7 of every step with the operators
of the fixed cloud, Sec. 3.2 and Sec. 5): (rho, U, T)^0 are the moments of
f^0, then ``nsteps`` steps, then the objective J(f, rho, U) of the final
state (lid heat flux plus weighted kinetic energy, see ``bgk_objective``).

``rollout_objective`` wraps it in a ``torch.autograd.Function``: the forward
pass keeps (f, U) every ``checkpoint_every`` steps; the backward pass walks
the segments in reverse, recomputes each segment's steps with
``bgk_step_keep``, which also keeps what the reverse step reads (f-tilde,
f^{n+1} and the new moments; about two f-sized arrays per step of the
segment), and runs ``bgk_adjoint_step_kept`` over them, accumulating dJ/dlid
on the device.  With ``keep_states=False`` the segment keeps only its
states and every ``bgk_adjoint_step`` recomputes its step (one f-sized
array per step, twice the forward work; the same gradients bit for bit).
The last segment, which the backward pass walks first, is run by the forward
pass in the same way where its arrays, with those of other such graphs,
take at most a quarter of the free device memory, and is not recomputed (3 steps of 48^3 x 20^3 FP32 in one
segment 151 -> 118 ms, 20 of 100^2 x 24^2 FP64 in two 11.1 -> 10.1).  They
stay allocated until the backward pass or the end of the graph; a program
that needs the memory in between turns this off with ``keep_states=False``,
under which nothing but the segment starts is held between the passes.
All arithmetic runs in libbgk; torch only holds the buffers.
"""
from __future__ import annotations

import threading
import weakref

import torch

from . import bgk as B
from .inputs import cloud_for


def segments(nsteps: int, every: int):
    """Checkpoint segments [(s0, s1), ...] covering steps 0..nsteps-1, in
    forward order; the state at s0 of each segment is stored."""
    if nsteps < 0 or every < 1:
        raise ValueError("nsteps >= 0 and checkpoint_every >= 1 are required")
    return [(s0, min(s0 + every, nsteps)) for s0 in range(0, nsteps, every)]


class _Kept(list):
    """The last segment's steps, from a forward pass to its backward."""

    __hash__ = object.__hash__  # (told apart by identity, for the set below)
    __eq__ = object.__eq__

    def __init__(self, steps, device, nbytes):
        super().__init__(steps)
        self.device, self.step_bytes = device, nbytes // len(steps)
        with _live_lock:
            _live.add(self)


_live, _live_lock = weakref.WeakSet(), threading.Lock()


def _held(device) -> int:
    """Bytes that the segments of all live graphs hold."""
    with _live_lock:
        return sum(len(k) * k.step_bytes for k in _live if k.device == device)


def _room(nbytes: int, device) -> bool:
    """Whether the last segment's arrays may stay allocated between a forward
    pass and its backward: together with those of other graphs at most a
    quarter of the memory free without them, so that graphs kept side by side
    stay within it and the backward pass, which needs as much again for a
    segment before it, has room.  Free is what the driver and the caching
    allocator together can hand out: the blocks of an earlier pass wait in
    the latter."""
    if torch.cuda.is_current_stream_capturing():
        return False
    held = _held(device)
    free = torch.cuda.mem_get_info(device)[0] + held
    if 4 * (nbytes + held) <= free:  # (the allocator's counters take 77 us to read)
        return True
    cached = torch.cuda.memory_reserved(device) - torch.cuda.memory_allocated(device)
    return 4 * (nbytes + held) <= free + cached


def _march(step, f, nsteps, every, *state):
    """nsteps calls step(f, f_next) from f, which is taken over; they advance
    ``state`` in place.  Returns the final f and {s: (f, *state)} of every
    segment start s (every None: of none)."""
    starts = {s0 for s0, _ in segments(nsteps, every)} if every else set()
    saved, spare = {}, None
    for s in range(nsteps):
        fn = torch.empty_like(f) if spare is None else spare
        spare = f
        if s in starts:
            saved[s] = (f, *(t.clone() for t in state))
            spare = None
        step(f, fn)
        f = fn
    return f, saved


def _tail(p, f0, nsteps, every, keep, fields):
    """Steps at the end of a rollout that the forward pass keeps for the
    backward, ``fields`` f-sized arrays each: the last segment, or none where
    no gradient is wanted, keep_states is off, there is no room, or the
    problem's own forward() has to be asked for the whole rollout."""
    own = getattr(p.forward, "__func__", None) not in _FORWARD
    if not keep or own or not p.keep_states or not every or nsteps <= 0:
        return 0
    s0, s1 = segments(nsteps, every)[-1]
    return s1 - s0 if _room((s1 - s0) * fields * f0.numel() * f0.element_size(),
                            p.ctx.device) else 0


class FrozenCavity:
    """A cavity on one GPU with a frozen cloud, set up for forward and reverse
    passes (BGK_FLAG_ADJOINT).  precision: "fp64", or "fp32" for FP32
    storage of f and of its adjoint (reductions stay FP64).  x: positions
    [d][N] of the frozen cloud (a torch tensor or numpy array; default the
    workload's initial cloud), e.g. where a moving-cloud run left it.
    keep_states: see the top of the file (False: least memory)."""

    def __init__(self, cav, device="cuda", seed=None, stream=None, precision="fp64", x=None,
                 keep_states=True, **overrides):
        if precision not in ("fp64", "fp32"):
            raise ValueError("the reverse mode runs in fp64 or fp32 storage")
        self.cav = cav
        self.keep_states = bool(keep_states)
        overrides = dict(overrides)
        overrides.update(move=0, flags=overrides.get("flags", 0) | B.BGK_FLAG_ADJOINT)
        self.cfg = B.config_from(cav, precision, **overrides)
        x0, wid = cloud_for(cav, seed)
        dev = torch.device(device)
        self.wall_id = torch.from_numpy(wid).to(dev)
        if x is None:
            self.x = torch.from_numpy(x0).to(dev)
        else:
            self.x = torch.as_tensor(x, dtype=torch.float64).to(dev).contiguous().clone()
            if tuple(self.x.shape) != tuple(x0.shape):
                raise ValueError(f"x must have shape {tuple(x0.shape)}")
        self.ctx = B.bgk_init(self.cfg, self.wall_id, stream)
        B.bgk_geometry(self.ctx, self.x)
        self.N, self.d, self.nc, self.NV = self.ctx.N, self.ctx.d, self.ctx.nc, self.ctx.NV

    def rest_state(self):
        """f^0 = M[1, 0, wall_T] at every particle (Chu: G1, G2)."""
        c = self.ctx
        rho = torch.ones(c.N, dtype=torch.float64, device=c.device)
        U = torch.zeros((c.d, c.N), dtype=torch.float64, device=c.device)
        T = torch.full((c.N,), float(self.cfg.wall_T), dtype=torch.float64, device=c.device)
        return B.bgk_maxwellian(c, rho, U, T)

    def forward(self, f0, lid, nsteps, every=None):
        """Run nsteps from f0 at lid speed ``lid``.  Returns the final state
        (f, rho, U, T) and the (f, U) stored at each segment start."""
        c = self.ctx
        B.bgk_set_lid_velocity(c, float(lid))
        # (a copy: by the time the backward pass reads f^0 the caller's storage
        # may have been written through its pointer, which autograd's version
        # counter does not see, and under saved-tensor hooks no version is
        # looked at; 110592 x 20^3 floats: 1.5 of 115 ms)
        f = f0.detach().clone()
        rho, U, T = B.bgk_moments(c, f)
        f, saved = _march(lambda f, fn: B.bgk_step(c, f, fn, self.x, U, rho, T), f, nsteps, every,
                          U)
        return (f, rho, U, T), saved

    def objective(self, f0, lid, nsteps, ke_weight=1.0):
        """J after nsteps (forward only; a float)."""
        (f, rho, U, _), _ = self.forward(f0, lid, nsteps)
        J = B.bgk_objective(self.ctx, f, rho, U, ke_weight, want_grad=False)
        return float(J.item())


def _kept_segment(p, fa, Ua, n):
    """n steps from (fa, Ua): [(f^n, U^n, (f-tilde, f, rho, U, T)^{n+1}), ...]."""
    steps = []
    for _ in range(n):
        fb, ft = torch.empty_like(fa), torch.empty_like(fa)
        Ub = Ua.clone()  # U^n in, U^{n+1} out
        rho, T = (torch.empty(p.N, dtype=torch.float64, device=fa.device) for _ in range(2))
        B.bgk_step_keep(p.ctx, fa, fb, p.x, Ub, rho, T, ft)
        steps.append((fa, Ua, (ft, fb, rho, Ub, T)))
        fa, Ua = fb, Ub
    return steps


def _states(step, fa, state, n):
    """The states before n steps from (fa, *state) by step(f, f_next, state),
    which advances state in place: [(f, *state), ...]."""
    states = [(fa, *state)]
    state = [t.clone() for t in state]
    for _ in range(n - 1):
        fb = torch.empty_like(fa)
        step(fa, fb, state)
        fa = fb
        states.append((fa, *(t.clone() for t in state)))
    return states


class _Rollout(torch.autograd.Function):
    @staticmethod
    def forward(actx, f0, lid, problem, nsteps, every, ke_weight, keep=False):
        p, c = problem, problem.ctx
        n = _tail(p, f0, nsteps, every, keep, 2)
        (f, rho, U, T), saved = p.forward(f0, lid, nsteps - n, every)
        last = None
        if n:
            saved[nsteps - n] = (f, U.clone())
            last = _Kept(_kept_segment(p, f, saved[nsteps - n][1], n), c.device,
                         2 * n * f.numel() * f.element_size())
            _, f, rho, U, _ = last[-1][2]
        J = B.bgk_objective(c, f, rho, U, ke_weight, want_grad=False)
        actx.problem, actx.nsteps, actx.every, actx.ke = problem, nsteps, every, ke_weight
        actx.final = (f, rho, U)
        actx.saved, actx.last = saved, last
        actx.lid = float(lid)
        actx.save_for_backward(f0)
        return J

    @staticmethod
    def backward(actx, gJ):
        (f0,) = actx.saved_tensors
        p, c = actx.problem, actx.problem.ctx
        B.bgk_set_lid_velocity(c, actx.lid)
        f, rho, U = actx.final
        _, (gf, grho, gU) = B.bgk_objective(c, f, rho, U, actx.ke, want_grad=True)
        g = gJ.to(torch.float64)
        lam_f, lam_U, lam_rho = gf.mul_(g), gU.mul_(g), grho.mul_(g)
        dlid = torch.zeros(1, dtype=torch.float64, device=c.device)
        first = True  # only the last step's rho, T feed the objective
        # the kept segment goes with its use (a second backward recomputes it)
        last, actx.last = actx.last if p.keep_states else None, None
        for s0, s1 in reversed(segments(actx.nsteps, actx.every)):
            fs, Us = actx.saved[s0]
            if p.keep_states:
                steps = _kept_segment(p, fs, Us, s1 - s0) if last is None else last
                last = None
                while steps:
                    fn, Un, kept = steps.pop()
                    B.bgk_adjoint_step_kept(c, fn, Un, p.x, kept, lam_f, lam_U,
                                            lam_rho if first else None, None, lam_f, lam_U, dlid)
                    first = False
                continue
            rho_t, T_t = torch.empty_like(rho), torch.empty_like(rho)
            states = _states(lambda f, fn, st: B.bgk_step(c, f, fn, p.x, st[0], rho_t, T_t),
                             fs, (Us,), s1 - s0)
            while states:
                fn, Un = states.pop()
                B.bgk_adjoint_step(c, fn, Un, p.x, lam_f, lam_U, lam_rho if first else None,
                                   None, lam_f, lam_U, dlid)
                first = False
        # (rho, U, T)^0 are the moments of f^0: U^0 enters the first step, and
        # with no steps rho^0 and U^0 enter J itself
        r0, U0, T0 = B.bgk_moments(c, f0)
        B.bgk_moments_adjoint(c, r0, U0, T0, lam_f, lam_rho if actx.nsteps == 0 else None,
                              lam_U, None)
        return lam_f, dlid.reshape(()), None, None, None, None, None


def _wanted(*inputs) -> bool:
    return torch.is_grad_enabled() and any(t.requires_grad for t in inputs)


def rollout_objective(problem: FrozenCavity, f0: torch.Tensor, lid: torch.Tensor, nsteps: int,
                      checkpoint_every: int = 10, ke_weight: float = 1.0) -> torch.Tensor:
    """J of the frozen-cloud rollout from f0 at lid speed ``lid`` (0-d float64
    tensor); differentiable in f0 and lid."""
    if not isinstance(lid, torch.Tensor):
        lid = torch.tensor(float(lid), dtype=torch.float64, device=f0.device)
    return _Rollout.apply(f0, lid, problem, int(nsteps), int(checkpoint_every), float(ke_weight),
                          _wanted(f0, lid))


class MovingCavity:
    """A cavity on one GPU whose cloud moves with the gas (S8), set up for
    forward and reverse passes through the positions (BGK_FLAG_ADJOINT,
    move = 1).  precision: "fp64" or "fp32" storage of f and its adjoint.
    keep_states: False holds no states from a forward pass to its backward
    but those at the segment starts."""

    keep_states = True

    def __init__(self, cav, device="cuda", seed=None, stream=None, precision="fp64",
                 keep_states=True, **overrides):
        if precision not in ("fp64", "fp32"):
            raise ValueError("the reverse mode runs in fp64 or fp32 storage")
        self.cav = cav
        self.keep_states = bool(keep_states)
        overrides = dict(overrides)
        overrides.update(move=1, flags=overrides.get("flags", 0) | B.BGK_FLAG_ADJOINT)
        self.cfg = B.config_from(cav, precision, **overrides)
        x, wid = cloud_for(cav, seed)
        dev = torch.device(device)
        self.wall_id = torch.from_numpy(wid).to(dev)
        self.x0 = torch.from_numpy(x).to(dev)
        self.ctx = B.bgk_init(self.cfg, self.wall_id, stream)
        self.N, self.d, self.nc, self.NV = self.ctx.N, self.ctx.d, self.ctx.nc, self.ctx.NV

    def rest_state(self):
        """f^0 = M[1, 0, wall_T] at every particle (Chu: G1, G2)."""
        c = self.ctx
        rho = torch.ones(c.N, dtype=torch.float64, device=c.device)
        U = torch.zeros((c.d, c.N), dtype=torch.float64, device=c.device)
        T = torch.full((c.N,), float(self.cfg.wall_T), dtype=torch.float64, device=c.device)
        return B.bgk_maxwellian(c, rho, U, T)

    def forward(self, f0, lid, nsteps, every=None, x0=None):
        """Run nsteps from (f0, x0) at lid speed ``lid``.  Returns the final
        state (f, rho, U, T, x) and the (f, U, x) stored at each segment
        start."""
        c = self.ctx
        B.bgk_set_lid_velocity(c, float(lid))
        f = f0.detach().clone()
        x = (self.x0 if x0 is None else x0).detach().clone()
        rho, U, T = B.bgk_moments(c, f)
        f, saved = _march(lambda f, fn: B.bgk_step(c, f, fn, x, U, rho, T), f, nsteps, every, U, x)
        return (f, rho, U, T, x), saved

    def objective(self, f0, lid, nsteps, ke_weight=1.0, x0=None):
        """J after nsteps (forward only; a float)."""
        (f, rho, U, _, _), _ = self.forward(f0, lid, nsteps, x0=x0)
        J = B.bgk_objective(self.ctx, f, rho, U, ke_weight, want_grad=False)
        return float(J.item())


# the forward passes that a rollout may cut short of its last segment
_FORWARD = (FrozenCavity.forward, MovingCavity.forward)


class _RolloutMove(torch.autograd.Function):
    @staticmethod
    def forward(actx, f0, lid, x0, problem, nsteps, every, ke_weight, keep=False):
        p, c = problem, problem.ctx
        n = _tail(p, f0, nsteps, every, keep, 1)
        (f, rho, U, T, x), saved = p.forward(f0, lid, nsteps - n, every, x0)
        last = None
        if n:
            saved[nsteps - n] = (f, U.clone(), x.clone())
            last = _Kept(_states(lambda f, fn, st: B.bgk_step(c, f, fn, st[1], st[0], rho, T),
                                 f, (U, x), n), c.device, n * f.numel() * f.element_size())
            fa, U, x = last[-1][0], last[-1][1].clone(), last[-1][2].clone()
            f = torch.empty_like(fa)
            B.bgk_step(c, fa, f, x, U, rho, T)
        J = B.bgk_objective(c, f, rho, U, ke_weight, want_grad=False)
        actx.problem, actx.nsteps, actx.every, actx.ke = problem, nsteps, every, ke_weight
        actx.final = (f, rho, U)
        actx.saved, actx.last = saved, last
        actx.lid = float(lid)
        actx.save_for_backward(f0)
        return J

    @staticmethod
    def backward(actx, gJ):
        (f0,) = actx.saved_tensors
        p, c = actx.problem, actx.problem.ctx
        B.bgk_set_lid_velocity(c, actx.lid)
        f, rho, U = actx.final
        _, (gf, grho, gU) = B.bgk_objective(c, f, rho, U, actx.ke, want_grad=True)
        g = gJ.to(torch.float64)
        lam_f, lam_U, lam_rho = gf.mul_(g), gU.mul_(g), grho.mul_(g)
        lam_x = torch.zeros_like(U)          # the objective does not read x
        dlid = torch.zeros(1, dtype=torch.float64, device=c.device)
        first = True  # only the last step's rho feeds the objective
        rho_t, T_t = torch.empty_like(rho), torch.empty_like(rho)
        # the kept segment goes with its use (a second backward recomputes it)
        states, actx.last = actx.last, None
        for s0, s1 in reversed(segments(actx.nsteps, actx.every)):
            if not states:
                fs, Us, xs = actx.saved[s0]
                states = _states(
                                 lambda f, fn, st: B.bgk_step(c, f, fn, st[1], st[0], rho_t, T_t),
                                 fs, (Us, xs), s1 - s0)
            while states:
                fn, Un, xn = states.pop()
                B.bgk_adjoint_step_move(c, fn, Un, xn, lam_f, lam_U, lam_x,
                                        lam_rho if first else None, None, lam_f, lam_U, lam_x,
                                        dlid)
                first = False
        r0, U0, T0 = B.bgk_moments(c, f0)
        B.bgk_moments_adjoint(c, r0, U0, T0, lam_f, lam_rho if actx.nsteps == 0 else None,
                              lam_U, None)
        return lam_f, dlid.reshape(()), lam_x, None, None, None, None, None


def rollout_objective_move(problem: MovingCavity, f0: torch.Tensor, lid: torch.Tensor,
                           nsteps: int, checkpoint_every: int = 10, ke_weight: float = 1.0,
                           x0: torch.Tensor | None = None) -> torch.Tensor:
    """J of the rollout with the moving cloud from (f0, x0) at lid speed
    ``lid``; differentiable in f0, lid and x0 (the initial positions, default
    the workload's cloud).  Checkpoints hold (f, U, x) every
    checkpoint_every steps; the backward pass recomputes each segment (the
    last one only where its states did not stay from the forward pass) and
    runs bgk_adjoint_step_move over it in reverse."""
    if not isinstance(lid, torch.Tensor):
        lid = torch.tensor(float(lid), dtype=torch.float64, device=f0.device)
    if x0 is None:
        x0 = problem.x0
    return _RolloutMove.apply(f0, lid, x0, problem, int(nsteps), int(checkpoint_every),
                              float(ke_weight), _wanted(f0, lid, x0))
