"""Gradient of the summed smooth KL sensor with respect to the initial velocity
field, by the library's hand-written adjoint kernels behind a
torch.autograd.Function, with checkpointing.

Loss: L(u0) = sum_x S_KL(g_N(x)), g_N the pre-collision populations of the
last of N D2Q9 steps started from the equilibrium of (rho0, u0) (the smooth
S_KL is sum_i f^eq_i phi(f^neq_i / f^eq_i), phi(x) = (1+x) ln(1+x) - x,
which equals the f term of eq. HKL-sensor).

Forward: N steps, keeping the state every `checkpoint` steps; only the last one
computes sensors.  Backward: for each checkpoint segment, newest first,
recompute its states, then run the reverse steps (seed at step N, then up to
three adjoint steps per launch) and finally the initial-condition adjoint.
Everything numeric runs in liblks.so; this module only orders the calls and
owns the buffers.
"""
import torch

from . import lks


# steps per launch of Lattice.trajectory and Lattice.adjoint_steps
_PER_LAUNCH = 3


def _advance(lat, src, dst, n, scratch):
    """n steps from src, the last state into dst; on the way only each launch's
    last state is stored, in the two scratch states in turn."""
    out = [None] * n
    for k, i in enumerate(range(_PER_LAUNCH - 1, n - 1, _PER_LAUNCH)):
        out[i] = scratch[k % 2]
    for i in range(n - n % _PER_LAUNCH, n - 1):
        # single steps at the end: each into the buffer that the one before left free
        out[i] = scratch[0] if out[i - 1] is not scratch[0] else scratch[1]
    out[n - 1] = dst
    lat.trajectory(src, out)


class _KLSensorLoss(torch.autograd.Function):
    @staticmethod
    def forward(ctx, ux0, uy0, rho0, tau, nsteps, checkpoint, dtype, layout):
        if nsteps < 1 or checkpoint < 1:
            raise ValueError("nsteps and checkpoint must be >= 1")
        ny, nx = ux0.shape
        dev = ux0.device
        lat = lks.Lattice(9, nx, ny, dtype, tau=tau, max_steps=nsteps, layout=layout, device=dev)
        lat.init(rho0, ux0.detach(), uy0.detach())
        ckpts = {0: lat.state.clone()}
        if lat.has_trajectory():
            # the loss needs the sensors of the last step only: the steps before
            # it advance the state alone, from checkpoint to checkpoint
            done = 0
            while done < nsteps - 1:
                m = min(checkpoint, nsteps - 1 - done)
                if m == checkpoint:
                    ckpts[done + m] = lat.new_state()
                    _advance(lat, ckpts[done], ckpts[done + m], m, lat.pop)
                else:
                    last = lat.new_state()
                    _advance(lat, ckpts[done], last, m, lat.pop)
                done += m
            lat.restore(ckpts[done] if done in ckpts else last, done)
            lat.step(1)
        else:
            done = 0
            while done < nsteps:
                m = min(checkpoint, nsteps - done)
                lat.step(m)
                done += m
                if done < nsteps:
                    ckpts[done] = lat.state.clone()
        loss = lat.sums[(nsteps - 1) % nsteps, 4].clone()
        ctx.lat = lat
        ctx.ckpts = ckpts
        ctx.meta = (nsteps, checkpoint)
        ctx.fields = [t.detach().to(dev, torch.float64).contiguous() for t in (rho0, ux0, uy0)]
        return loss

    @staticmethod
    def backward(ctx, grad_out):
        lat, ckpts = ctx.lat, ctx.ckpts
        nsteps, K = ctx.meta
        rho0, ux0, uy0 = ctx.fields
        seg = [lat.new_state() for _ in range(min(K, nsteps) - 1)]
        lam = [lat.new_state() for _ in range(2)]
        cur = 0                      # lam[cur] holds dL/dg_{n+1} entering step n
        several = lat.has_trajectory()
        for s in sorted(ckpts, reverse=True):
            e = min(s + K - 1, nsteps - 1)          # states f_s .. f_e
            states = [ckpts[s]] + seg[: e - s]
            if several:
                lat.trajectory(states[0], states[1:])
            else:
                for j in range(1, e - s + 1):
                    lat.step_from(states[j - 1], states[j])
            n = e + 1                               # reverse steps n = e+1 .. s+1
            if n == nsteps:
                lat.adjoint_seed_kl(states[n - 1 - s], lam[cur])
                n -= 1
            while n > s:
                m = min(_PER_LAUNCH, n - s) if several else 1
                lat.adjoint_steps([states[n - j - 1 - s] for j in range(m)], lam[cur], lam[1 - cur])
                cur = 1 - cur
                n -= m
        gux = torch.empty_like(ux0)
        guy = torch.empty_like(uy0)
        lat.adjoint_init(rho0, ux0, uy0, lam[cur], gux, guy)
        g = grad_out.to(torch.float64)
        return gux * g, guy * g, None, None, None, None, None, None


def kl_sensor_loss(ux0, uy0, rho0, tau=0.52, nsteps=200, checkpoint=20, dtype="f32",
                   layout="planes"):
    """L = sum of the smooth KL sensor at the last of nsteps steps (0-dim
    float64 tensor), differentiable w.r.t. ux0 and uy0 ([ny, nx] float64 CUDA
    tensors); rho0 is held fixed.  layout: the population layout of the
    states the forward and reverse steps run on."""
    return _KLSensorLoss.apply(ux0, uy0, rho0, tau, nsteps, checkpoint, dtype, layout)
