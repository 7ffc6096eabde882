"""Gradients of plane-statistics losses by the library's discrete adjoint step.

The forward run keeps the states and inlet planes of its last steps, as many
as KEEP_SHARE of the device memory that the run would leave free without them
holds (lbm_step_keep), and before them, or with `segment` given throughout, the
state every `segment` steps (default about sqrt(T)).  So a run takes memory in
proportion to sqrt(T) with `segment` given, and up to KEEP_SHARE of the free
memory more without, from its first forward run on for as long as it lives.  The backward sweep runs lbm_adjoint_step backwards through the
kept states and recomputes each segment from its checkpoint into a ring of
state buffers (lbm_step_record, which also keeps each step's inlet plane).
Every step of both sweeps runs in the library's kernels; this module only
orders the calls and holds the buffers.

    run = StatsGradient(ch, planes=[128], nsteps=400)
    means = plane_statistics(run, amp_bin, cs)   # torch.autograd.Function
    loss = mean_profile_loss(means[0], U_target, R12_target)
    loss.backward()                              # amp_bin.grad, cs.grad
"""
import math

import numpy as np
import torch


# Share of the device memory free at the first forward run, less what the run
# takes besides, that the kept states may take.  A kept step saves its recompute:
# 256 x 64 x 64, 30 steps, forward and sweep 3.61 -> 2.68 ms.  The rest stays for
# the program.
KEEP_SHARE = 1 / 8


class StatsGradient:
    """Forward statistics run and adjoint gradient sweep on one Channel.

    The channel's current state at construction is the initial state s_0 of
    every run.  Statistics are the means over z and steps 1..nsteps at the x
    planes given (lbm_stats); the gradient is taken with respect to the STG
    amplitude scalings s_b and C_s.
    """

    def __init__(self, ch, planes, nsteps, segment=None):
        self.ch = ch
        self.planes = [int(p) for p in planes]
        self.T = int(nsteps)
        self.seg = int(segment) if segment else max(1, int(round(math.sqrt(self.T))))
        f, h = ch.state()
        self.t0 = ch.time
        self.f0 = f.clone()
        self.h0 = h.clone()
        self.ckpt = []
        self._auto = not segment
        self._ring = self._lam = self._kept = None

    def _keep_states(self):
        """Number of states that fit KEEP_SHARE of the device memory that is free beside the
        checkpoints, the recompute ring and the adjoint fields of a run without kept states."""
        dev = self.f0.device
        free = torch.cuda.mem_get_info(dev)[0] + torch.cuda.memory_reserved(dev) - torch.cuda.memory_allocated(dev)
        state = self.f0.nbytes + self.h0.nbytes + 6 * 4 * self.ch.ny * self.ch.nz
        need = (-(-self.T // self.seg) + max(self.seg - 1, 1)) * state + 2 * (4 * self.f0.numel() + self.h0.nbytes)
        return max(0, int(KEEP_SHARE * (free - need)) // state)

    def _keep(self):
        """Buffers of the kept steps: n states and n + 1 inlet planes (of no step: n = 0)."""
        if self._kept is None:
            n = min(self.T - 1, self._keep_states()) if self._auto else 0
            size = -(-self.f0.numel() // 128) * 128  # states begin on 256-byte borders
            dev, plane = self.f0.device, (n + 1, 3, self.ch.ny, self.ch.nz)
            try:
                f = torch.empty(n * size, dtype=self.f0.dtype, device=dev)
                h = torch.empty((n,) + tuple(self.h0.shape), dtype=torch.float32, device=dev)
                u, fl = (torch.empty(plane if n else (0,), dtype=torch.float32, device=dev) for _ in range(2))
            except torch.cuda.OutOfMemoryError:
                n = 0
            if n < 1:
                self._kept = dict(f=[], h=[], u=[], fl=[])
            else:
                f = [f[k * size:k * size + self.f0.numel()].view(self.f0.shape) for k in range(n)]
                self._kept = dict(f=f, h=list(h.unbind(0)), u=list(u.unbind(0)), fl=list(fl.unbind(0)))
                torch.cuda.current_stream(dev).synchronize()  # the channel may run on another stream
        return self._kept

    def forward(self):
        """Run nsteps from s_0 with statistics; returns the means [n_planes, ny, 9] (float64 numpy)."""
        ch = self.ch
        ch.set_state(self.f0, self.h0, self.t0)
        ch.stats_attach(self.planes)
        self.ckpt = []
        kept = self._keep()
        n_kept = len(kept["u"])
        k = 0
        while k < self.T - n_kept:
            f, h = ch.state()
            self.ckpt.append((f.clone(), h.clone(), ch.time))
            n = min(self.seg, self.T - n_kept - k)
            ch.step(n)
            k += n
        if n_kept:
            start = tuple(t.clone() for t in ch.state()) if k else (self.f0, self.h0)
            self.ckpt.append(start + (ch.time,))
            ch.step_keep(n_kept, kept["f"], kept["h"], kept["u"], kept["fl"])
        means, n = ch.stats_read()
        assert n == self.T, (n, self.T)
        return means

    def _buffers(self):
        ch = self.ch
        f, h = ch.state()
        if self._lam is None:
            self._lam = [ch.new_field(), ch.new_field()]
            self._eta = [torch.zeros_like(h), torch.zeros_like(h)]
        if self._ring is None and self.T > len(self._keep()["u"]):
            n = max(self.seg - 1, 1)
            plane = (3, ch.ny, ch.nz)
            self._ring = dict(f=[torch.empty_like(f) for _ in range(n)], h=[torch.empty_like(h) for _ in range(n)],
                              u=[torch.empty(plane, dtype=torch.float32, device=ch.device) for _ in range(n)],
                              fl=[torch.empty(plane, dtype=torch.float32, device=ch.device) for _ in range(n)])
        return self._ring

    def backward(self, dmeans, time_kernel=False):
        """Gradient from dL/dmeans [n_planes, ny, 9]: returns float64 numpy [n_bins + 1]
        (dL/ds_b..., dL/dC_s).  With time_kernel, also the summed time of the adjoint steps in ms
        (HIP events around each segment's adjoint steps)."""
        ch = self.ch
        ring = self._buffers()
        ch.stats_detach()  # the sampled planes keep their kernel: the recompute matches the forward run bit for bit
        open_ = ch.cfg.xbc == 1
        # each step adds one z-sum per (plane, y) to the accumulators; means divide by nz T
        coef = torch.as_tensor(np.asarray(dmeans, dtype=np.float64) / (ch.nz * self.T), dtype=torch.float32,
                               device=ch.device).contiguous()
        n_bins = 0 if ch._stg is None else int(ch._stg.n_bins)
        grad = torch.zeros(n_bins + 1, dtype=torch.float64, device=ch.device)
        lam, eta = self._lam, self._eta
        for t in lam + eta:
            t.zero_()
        ev = []
        t_last = self.t0 + 1  # the sweep's last adjoint step reduces the parameter gradient
        kept = self._keep()
        t_kept = self.t0 + self.T - len(kept["u"])  # the kept steps are those from here on
        for f_k, h_k, t_k in reversed(self.ckpt):
            if t_k >= t_kept:
                L, buf, n_planes = len(kept["u"]), kept, len(kept["u"])
            else:
                L, buf = min(self.seg, t_kept - t_k), ring
                n_planes = L - 1
                # recompute s_{t_k + j}, j = 1 .. L-1, and the inlet planes of those steps
                if L > 1:
                    ch.step_record(f_k, h_k, t_k, ring["f"][:L - 1], ring["h"][:L - 1],
                                   ring["u"][:L - 1] if open_ else None, ring["fl"][:L - 1] if open_ else None)
            states = [f_k] + buf["f"][:L - 1]
            hists = [h_k] + buf["h"][:L - 1]
            if time_kernel:
                e0 = torch.cuda.Event(enable_timing=True)
                e1 = torch.cuda.Event(enable_timing=True)
                e0.record()
            for j in reversed(range(L)):
                has_plane = open_ and j < n_planes  # the plane of step j was kept
                ch.adjoint_step(states[j], hists[j], t_k + j + 1, lam[0], lam[1], eta[0], eta[1], coef=coef,
                                grad=grad if t_k + j + 1 == t_last else None,
                                u_in=buf["u"][j] if has_plane else None, fluct=buf["fl"][j] if has_plane else None)
                lam.reverse()
                eta.reverse()
            if time_kernel:
                e1.record()
                ev.append((e0, e1))
        ch.point_state(ch.f[0], ch.f[1], ch.hist[0], ch.hist[1], self.t0)
        ch.set_state(self.f0, self.h0, self.t0)
        ch.sync()
        g = grad.cpu().numpy()
        if time_kernel:
            return g, sum(a.elapsed_time(b) for a, b in ev)
        return g


class _PlaneStatistics(torch.autograd.Function):
    @staticmethod
    def forward(ctx, amp_bin, cs, run):
        run.ch.set_amp_bin(amp_bin.detach().cpu().numpy())
        run.ch.set_cs_smag(float(cs))
        ctx.run = run
        return torch.as_tensor(run.forward(), dtype=torch.float64)

    @staticmethod
    def backward(ctx, gmeans):
        g = ctx.run.backward(gmeans.detach().cpu().numpy())
        return torch.as_tensor(g[:-1]), torch.as_tensor(g[-1]), None


def plane_statistics(run, amp_bin, cs):
    """Means [n_planes, ny, 9] of (u, v, w, uu, vv, ww, uv, uw, vw) as a differentiable
    function of the amplitude scalings amp_bin [n_bins] and C_s (float64 CPU tensors)."""
    return _PlaneStatistics.apply(amp_bin, cs, run)


def mean_profile_loss(means, U_target, R12_target):
    """sum_y (U - U_t)^2 / sum U_t^2 + sum_y (<u'v'> - R12)^2 / sum R12^2 for one plane's
    means [ny, 9], <u'v'> = <uv> - <u><v>."""
    U_target = torch.as_tensor(U_target, dtype=torch.float64)
    R12_target = torch.as_tensor(R12_target, dtype=torch.float64)
    U, V, UV = means[:, 0], means[:, 1], means[:, 6]
    uv = UV - U * V
    return ((U - U_target) ** 2).sum() / (U_target ** 2).sum() + ((uv - R12_target) ** 2).sum() / (R12_target ** 2).sum()
