"""Differentiable DUGKS rollout: torch.autograd.Function over the library's
forward step, hand-written adjoint step, initial-state VJP and read-out VJP,
with sqrt(N) checkpointing (Griewank-style two-level recomputation).

Memory: ceil(sqrt(N)) checkpoint states plus one segment of at most
ceil(sqrt(N)) states during the backward pass; compute: one extra forward
pass.  Any mesh and boundary set of the incompressible model (those of the
adjoint step).
"""
from __future__ import annotations

import math

import torch

from . import (_VP, _check, _ptr, _stream, dugks_destroy, dugks_init, dugks_init_vjp, dugks_moments,
               dugks_moments_vjp, dugks_run, dugks_step, load, shape_of)


class _Rollout(torch.autograd.Function):
    @staticmethod
    def forward(actx, force, u0, cfg, nsteps, seg):
        Q, D, shp = shape_of(cfg)
        dt = float(cfg["dt"])
        f = torch.empty((Q,) + shp, dtype=force.dtype, device=force.device)
        h = dugks_init(cfg, f, None, u0, force)
        # a segment at a time, out of place from its checkpoint; two calls each
        # (a call per step costs the host more than a step takes on the device)
        ckpt = {0: f}
        spare = torch.empty_like(f)
        n = 0
        while n < nsteps:
            m = min(seg, nsteps - n)
            g = torch.empty_like(f)
            dugks_step(h, f, g, force, n * dt)
            if m > 1 and dugks_run(h, g, spare, m - 1, force, (n + 1) * dt):
                g, spare = spare, g
            f = g
            n += m
            if n < nsteps:
                ckpt[n] = f
        u = torch.empty((D,) + shp, dtype=force.dtype, device=force.device)
        dugks_moments(h, f, force, nsteps * dt, None, u, None, totals=False)
        actx.h, actx.cfg, actx.nsteps, actx.seg, actx.ckpt = h, cfg, nsteps, seg, ckpt
        actx.save_for_backward(force, u0)
        return u

    @staticmethod
    def backward(actx, grad_u):
        force, u0 = actx.saved_tensors
        h, cfg, nsteps, seg, ckpt = actx.h, actx.cfg, actx.nsteps, actx.seg, actx.ckpt
        dt = float(cfg["dt"])
        Q, D, shp = shape_of(cfg)
        grad_u = grad_u.contiguous()
        gforce = torch.zeros_like(force)
        lam = torch.empty((Q,) + shp, dtype=force.dtype, device=force.device)
        lam2 = torch.empty_like(lam)
        dugks_moments_vjp(h, lam, None, grad_u, nsteps * dt, gforce)
        starts = sorted(ckpt.keys())
        # one segment's states, recomputed step by step straight into their
        # slots (slot 0 is the checkpoint itself)
        seg_states = torch.empty((seg - 1, Q) + shp, dtype=force.dtype, device=force.device) if seg > 1 else None
        # the library's entry points with their arguments converted once: through
        # the checked wrappers a call took the host 9 to 11 us, longer than the
        # device takes for a small mesh's step
        lib = load()
        step, adjoint, hp, st = lib.dugks_step, lib.dugks_step_adjoint, _VP(h), _stream(None)
        fp, gp = _ptr(force), _ptr(gforce)
        slots, nbytes = seg_states.data_ptr() if seg > 1 else 0, lam.numel() * lam.element_size()

        def call(fn, *args):
            rc = fn(*args)
            if rc:
                _check(rc, hp)

        for s0 in reversed(starts):
            s1 = min(s0 + seg, nsteps)

            def state(n):
                return ckpt[s0].data_ptr() if n == s0 else slots + (n - s0 - 1) * nbytes

            for n in range(s0, s1 - 1):
                call(step, hp, state(n), state(n + 1), fp, n * dt, st)
            for n in reversed(range(s0, s1)):
                call(adjoint, hp, state(n), fp, n * dt, lam.data_ptr(), lam2.data_ptr(), gp, st)
                lam, lam2 = lam2, lam
        gu0 = torch.zeros_like(u0)
        dugks_init_vjp(h, lam, u0, force, 0.0, gu0, gforce)
        dugks_destroy(h)
        actx.h = None
        return gforce, gu0, None, None, None


def rollout(cfg: dict, force: torch.Tensor, u0: torch.Tensor, nsteps: int, segment: int | None = None):
    """Final velocity u(t_N) [D, nz, ny, nx] after nsteps from the equilibrium
    state at (rho0, u0) under the force field `force`; differentiable in
    force and u0.  segment: steps between two checkpoints, at least 1 (None or
    0: ceil(sqrt(nsteps)))."""
    seg = int(segment or max(1, math.ceil(math.sqrt(nsteps))))
    if seg < 1:
        raise ValueError("segment must be at least 1")
    return _Rollout.apply(force.contiguous(), u0.contiguous(), dict(cfg), int(nsteps), seg)
