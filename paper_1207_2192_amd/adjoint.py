"""Hand-written adjoint of RK4 and Heun trajectories as a torch.autograd.Function.

`CoreTrajectory.apply(m0, alpha, c, disk, params, n_seg, seg_steps, lambda_ex_nm, noise)`
integrates n_seg * seg_steps RK4 steps (noise = None) or Heun steps (noise =
(seed, step0, replica); segment s uses the step indices step0 + s*seg_steps ...)
on the GPU and returns the vortex core position r_c (nm, float64) at the
n_seg + 1 checkpoints t = 0, seg_steps, ...  Checkpoints of the state are kept
every seg_steps steps.  Where a gradient is asked for, the forward pass steps with
the stage record (llg_rk4_record / llg_heun_record) and keeps it for as many
segments as RECORD_SHARE of the device's memory holds beside those of the other
trajectories that wait for theirs (5000 RK4 steps at R = 80 nm: 3 GB of 288); the
backward pass recomputes the record of the others from their checkpoints.  It
runs the reverse sweep (llg_rk4_vjp / llg_heun_vjp, the noise replayed from its
counter); the cotangent of each sampled core position enters through
llg_core_position_vjp.
Gradients come out for m0, alpha and c = a^2/lambda_ex^2;
`grad_exchange_length` converts d/dc into d/d lambda_ex.  All arithmetic runs
in lib_llgdisk; torch provides buffers and the stream.
"""
from __future__ import annotations

import threading
from dataclasses import replace

import torch

from ._lib import STEP_COUNTER
from .api import Disk, LLGParams


# Records are kept between the passes, by all trajectories of the process together, up
# to RECORD_SHARE of the device's memory (18 GB of 288), and by one up to FREE_SHARE of
# what is free.  A recorded RK4 step costs 36.3 us against 35.7 plain at R = 80 nm (17.1
# against 16.3 at 30 nm), so recomputing a segment is a whole forward pass over: 2 x 50
# steps at R = 80 nm, forward and backward, 13.5 ms recomputed and 10.2 ms kept.
RECORD_SHARE = 1.0 / 16
FREE_SHARE = 1.0 / 8


class _Record:
    """A segment's record, counted against the device's share until it is dropped."""
    held: dict = {}                 # bytes kept, by device
    lock = threading.RLock()        # taken again by a drop that a collection inside it causes

    def __init__(self, floats: int, device):
        self.device, self.bytes = device, 0
        self.data = torch.empty(floats, dtype=torch.float32, device=device)
        self.bytes = 4 * floats
        with self.lock:
            self.held[device] = self.held.get(device, 0) + self.bytes

    def __del__(self):
        with self.lock:
            self.held[self.device] = self.held.get(self.device, 0) - self.bytes


def _kept_segments(n_seg: int, seg_floats: int, device) -> int:
    """Segments whose record the forward pass may keep until the backward pass."""
    free, total = torch.cuda.mem_get_info(device)
    with _Record.lock:
        room = min(RECORD_SHARE * total - _Record.held.get(device, 0), FREE_SHARE * free)
    return max(0, min(n_seg, int(room // (4 * max(seg_floats, 1)))))


def _take_records(segments, seg_floats: int, device) -> dict:
    """Memory for the records of the last of the given segments, as many as may be kept."""
    out = {}
    with _Record.lock:
        keep = _kept_segments(len(segments), seg_floats, device)
        for s in segments[len(segments) - keep:][::-1]:
            try:
                out[s] = _Record(seg_floats, device)
            except torch.OutOfMemoryError:      # held by others in the meantime
                break
    return out


def _record_floats(disk: Disk, seg_steps: int, noise) -> int:
    return (8 if noise is None else 4) * seg_steps * disk.state_size


def _explicit_steps(noise, s: int, seg_steps: int) -> bool:
    """Whether segment s can be recorded: a first step index that is STEP_COUNTER as 64
    bits stands for the handle's counter, which plain steps take and a record does not."""
    return noise is None or (int(noise[1]) + s * seg_steps) % 2 ** 64 != STEP_COUNTER


def _record(disk: Disk, m, seg_steps: int, prm, noise, s: int, rec):
    """Segment s of the trajectory in place, with its stage record."""
    if noise is None:
        disk.rk4_record(m, seg_steps, prm, rec)
    else:
        seed, step0, rep = noise
        disk.heun_record(m, seg_steps, prm, rec, seed=seed, step0=step0 + s * seg_steps, replica=rep)


class CoreTrajectory(torch.autograd.Function):
    @classmethod
    def apply(cls, *args):
        # forward always runs with gradients off, so the caller's mode goes along: without gradients no
        # backward pass can follow, and nothing is recorded
        noise = (None,) if len(args) == 8 else ()
        return super().apply(*args, *noise, torch.is_grad_enabled())

    @staticmethod
    def forward(ctx, m0, alpha, c, disk: Disk, params: LLGParams, n_seg: int, seg_steps: int,
                lambda_ex_nm: float, noise, grad_enabled: bool):
        if disk.n != 1:
            raise ValueError("CoreTrajectory steps one disk")
        if noise is None and params.renorm:
            raise ValueError("the RK4 adjoint covers RK4 without renormalisation")
        prm = replace(params, alpha=float(alpha), c=float(c))
        m = m0.detach().clone().contiguous()
        ckpts = [m.clone()]
        cores = [disk.vortex_core_position(m, lambda_ex_nm)]
        recs = {}
        if grad_enabled and any(ctx.needs_input_grad) and seg_steps > 0:
            recs = _take_records([s for s in range(n_seg) if _explicit_steps(noise, s, seg_steps)],
                                 _record_floats(disk, seg_steps, noise), m.device)
        for s in range(n_seg):
            if s in recs:
                _record(disk, m, seg_steps, prm, noise, s, recs[s].data)
            elif noise is None:
                disk.rk4_step(m, seg_steps, prm)
            else:
                seed, step0, rep = noise
                disk.heun_step(m, seg_steps, prm, seed=seed, step0=step0 + s * seg_steps, replica=rep)
            ckpts.append(m.clone())
            cores.append(disk.vortex_core_position(m, lambda_ex_nm))
        ctx.noise, ctx.recs = noise, recs
        ctx.disk, ctx.prm, ctx.n_seg, ctx.seg = disk, prm, n_seg, seg_steps
        ctx.lam, ctx.ckpts, ctx.cores = lambda_ex_nm, ckpts, cores
        ctx.alpha_like, ctx.c_like = alpha, c
        return torch.stack([cr[0, :2] for cr in cores])

    @staticmethod
    def backward(ctx, grad_rc):
        disk, prm, seg = ctx.disk, ctx.prm, ctx.seg
        grad_rc = grad_rc.to(torch.float64).contiguous()
        ybar = torch.zeros_like(ctx.ckpts[0])
        pgrad = torch.zeros(2, dtype=torch.float64, device=ybar.device)
        rec = None
        disk.core_position_vjp(ctx.ckpts[-1], ctx.lam, ctx.cores[-1], grad_rc[-1], ybar)
        for s in reversed(range(ctx.n_seg)):
            kept = ctx.recs.pop(s, None)                  # given back once read; a second backward pass recomputes it
            if kept is not None:
                cur = kept.data
            else:
                if rec is None:
                    rec = torch.empty(_record_floats(disk, seg, ctx.noise), dtype=torch.float32, device=ybar.device)
                cur = rec
                _record(disk, ctx.ckpts[s].clone(), seg, prm, ctx.noise, s, cur)
            if ctx.noise is None:
                disk.rk4_vjp(cur, seg, ybar, pgrad, prm)
            else:
                seed, step0, rep = ctx.noise
                disk.heun_vjp(cur, seg, ybar, pgrad, prm, seed=seed, step0=step0 + s * seg, replica=rep)
            disk.core_position_vjp(ctx.ckpts[s], ctx.lam, ctx.cores[s], grad_rc[s], ybar)
        ga = pgrad[0].to(dtype=torch.as_tensor(ctx.alpha_like).dtype)
        gc = pgrad[1].to(dtype=torch.as_tensor(ctx.c_like).dtype)
        if isinstance(ctx.alpha_like, torch.Tensor):
            ga = ga.to(ctx.alpha_like.device)
        if isinstance(ctx.c_like, torch.Tensor):
            gc = gc.to(ctx.c_like.device)
        return ybar, ga, gc, None, None, None, None, None, None, None


def core_trajectory(m0, alpha, c, disk, params, n_seg, seg_steps, lambda_ex_nm, noise=None):
    """noise = None: RK4; noise = (seed, step0, replica): Heun with that Philox stream."""
    return CoreTrajectory.apply(m0, alpha, c, disk, params, n_seg, seg_steps, lambda_ex_nm, noise)


def grad_exchange_length(grad_c, c, lambda_ex_nm):
    """d/d lambda_ex from d/dc with c = (a/lambda_ex)^2: dc/dlambda = -2c/lambda."""
    return grad_c * (-2.0 * c / lambda_ex_nm)
