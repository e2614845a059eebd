"""Differentiable time loop: soma voltage traces of an implicit-Euler
simulation as a function of the edge conductances a, the capacitive terms c
and the injected currents I, with a hand-written adjoint.

Forward (paper §1, the current evaluated at the old step):
    A V^k = c V^{k-1} + I,  V^0 = 0,  A = diag(c) + L(a),  k = 1 .. steps,
    traces[k-1, cell] = V^k at the cell's root.
Backward, given G[k-1, cell] = dLoss/dtraces[k-1, cell]; A is symmetric, so
each adjoint step is one more solve with the same matrix:
    lambda^{steps+1} = 0;  for k = steps .. 1:
        A lambda^k = c lambda^{k+1} + G[k-1] at the roots
        dL/dI   += lambda^k
        dL/dc_i += lambda^k_i (V^{k-1}_i - V^k_i)
        dL/da_i += -(lambda^k_i - lambda^k_p)(V^k_i - V^k_p),  p = parent(i)
States are checkpointed every ``checkpoint_every`` steps and recomputed one
segment at a time during the backward pass; the kernels are deterministic,
so the recomputed states equal the forward ones bit for bit.

All arithmetic runs in the library's kernels (hines_assemble, hines_run_steps,
hines_adjoint_steps, hines_adjoint_accumulate_steps); torch provides the device
buffers.
"""
from __future__ import annotations

import torch

# adjoint steps between two accumulations: bounds the adjoint states kept at a
# time whatever the checkpoint distance (16 steps of a launch against 10 or 100
# differ by the first step's elimination, a few percent)
ADJOINT_ROWS = 16


class _SomaTraces(torch.autograd.Function):
    @staticmethod
    def forward(ctx, a, c, I, plan, steps, checkpoint_every):
        a = a.contiguous()
        c = c.contiguous()
        I = I.contiguous()
        diag, upper = plan.assemble(a, c)
        V = torch.zeros_like(c)
        traces = torch.empty(steps, plan.ncells, dtype=torch.float64, device=c.device)
        ckpts = [V]
        for k0 in range(0, steps, checkpoint_every):
            k1 = min(k0 + checkpoint_every, steps)
            nxt = torch.empty_like(c)
            plan.run_steps(diag, upper, c, V, k1 - k0, i_inj=I, v_out=nxt, traces=traces[k0:k1])
            V = nxt
            if k1 < steps:
                ckpts.append(V)
        ctx.plan = plan
        ctx.steps = steps
        ctx.every = checkpoint_every
        ctx.save_for_backward(c, I, diag, upper, *ckpts)
        return traces

    @staticmethod
    def backward(ctx, G):
        plan, steps, every = ctx.plan, ctx.steps, ctx.every
        c, I, diag, upper, *ckpts = ctx.saved_tensors
        G = G.contiguous()
        ga = torch.zeros_like(c)
        gc = torch.zeros_like(c)
        gi = torch.zeros_like(c)
        n = c.numel()
        states_buf = torch.empty(min(every, steps), n, dtype=c.dtype, device=c.device)
        lams_buf = torch.empty(min(every, steps, ADJOINT_ROWS), n, dtype=c.dtype, device=c.device)
        lam = None
        nseg = (steps + every - 1) // every
        for s in range(nseg - 1, -1, -1):
            k0 = s * every
            k1 = min(k0 + every, steps)
            states = states_buf[:k1 - k0]
            plan.run_steps(diag, upper, c, ckpts[s], k1 - k0, i_inj=I, states=states)
            for e in range(k1, k0, -ADJOINT_ROWS):
                b = max(e - ADJOINT_ROWS, k0)
                lams = lams_buf[:e - b]
                plan.adjoint_steps(diag, upper, c, lam, G[b:e], lams)
                v0 = ckpts[s] if b == k0 else states[b - k0 - 1]
                plan.adjoint_accumulate_steps(lams, states[b - k0:e - k0], v0, ga, gc, gi)
                lam = lams[0].clone()
        return ga, gc, gi, None, None, None


def soma_traces(plan, a, c, I, steps: int, checkpoint_every: int = 10):
    """Soma voltages [steps, ncells] of the simulation, differentiable w.r.t.
    a (edge conductance stored at the child; roots ignored), c and I.  The
    backward pass holds the states of ``checkpoint_every`` steps (its sign is
    ignored) and the adjoints of up to ``ADJOINT_ROWS`` of them at a time."""
    every = abs(int(checkpoint_every))
    if every == 0 and steps > 0:
        raise ValueError("checkpoint_every must not be 0")
    return _SomaTraces.apply(a, c, I, plan, int(steps), max(every, 1))
