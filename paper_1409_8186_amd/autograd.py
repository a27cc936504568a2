"""torch.autograd.Function around mudiff_grad: the far-field misfit of B disk
clusters as a differentiable function of their centers, radii and wavenumbers.

The forward pass rebuilds the device tables from the current parameters (the
Hankel tables are recomputed, not stored across calls), runs the forward and
adjoint solves in mudiff_grad and keeps the gradient; backward scales it by
the incoming gradient of each instance's loss.  Truncation orders N_p are
fixed inputs (not differentiated).
"""
from __future__ import annotations

import numpy as np
import torch

from . import _lib as L
from .api import Problem


def _misfit_grad(inst, device, betas, thetas, target, opts):
    """Problem.grad of the instances, in the form and with the solver that suit the columns."""
    R = (betas if isinstance(betas, torch.Tensor) else np.asarray(betas)).reshape(len(inst), -1).shape[1]
    restart = opts.get("restart", 50)
    circulant, sstep = opts.get("circulant"), opts.get("sstep")
    disks = [len(n) for _, _, n, _ in inst]
    orders_ok = max(int(np.max(n)) for _, _, n, _ in inst) <= 31  # else no apply on the matrix cores
    unknowns = sum(2 * int(np.sum(n)) + len(n) for _, _, n, _ in inst) / len(inst)  # of a column
    # The circulant form carries the solves of 8 and more columns, but for instances so small
    # that its transforms cost what it saves (ms a gradient, direct and circulant form: 100 disks
    # of order 31, 64 columns 257, 54; 30 of order 4, 8 columns 13.4, 11.7; 16 x 10 of order 31 9.7,
    # 6.1; 4 x 10 of orders 13..20 9.7, 11.3; 200 x 3 of order 4 3.4, 3.7).  Its tables are two to
    # three times the direct form's, so where they do not fit the direct form solves alone.
    auto_circulant = circulant is None
    if auto_circulant:
        circulant = R >= 8 and orders_ok and (max(disks) >= 24 or (max(disks) >= 10 and sum(disks) >= 128))
    # s-step solves (restarts of 20 to 64) halve the basis sweeps of long solves of long columns,
    # and take the host 6 to 20 us a column for their shifts (ms a gradient, one-vector and s-step
    # solves: 4 x 100 disks of order 4, 64 columns 118, 102; 60 of order 31, 64 columns 35, 30; 16 x 30
    # of order 31, 16 columns 32, 29, of order 4 19.1, 19.6; 32 x 16 of order 31, 64 columns 79, 101;
    # 200 x 3 of order 4 10, 261).  Where one stagnates, one-vector cycles solve.
    auto_sstep = sstep is None
    if auto_sstep:
        mean = sum(disks) / len(inst)
        long = mean >= 50 or (mean >= 24 and unknowns >= 1500)
        sstep = 10 if R >= 8 and orders_ok and long and 20 <= restart <= 64 else 0
    while True:
        P = None
        try:
            P = Problem(inst, device=device, circulant=circulant)
            return P.grad(betas, thetas, target, restart=restart, tol=opts.get("tol", 1e-10),
                          maxit=opts.get("maxit", 20000), flags=L.SSTEP | L.sstep_size(sstep) if sstep else 0)
        except torch.OutOfMemoryError:
            if not (auto_circulant and circulant or auto_sstep and sstep):
                raise
            circulant = circulant and not auto_circulant
            sstep = 0 if auto_sstep else sstep
        except L.MudiffError as e:
            if L.STATUS.get(e.status) != "NOT_CONVERGED" or not (auto_sstep and sstep):
                raise
            sstep = 0
        finally:
            if P is not None:
                P.close()


class FarFieldMisfit(torch.autograd.Function):
    """loss[b] = sum_{r, j} |a_b(theta_j; beta_{b,r}) - target_{b,r,j}|^2.

    Arguments: centers [M,2] float64, radii [M] float64, k [B] float64 (the
    differentiable inputs), then n_modes [M] (int), disk_off [B+1] (int),
    betas [B,R], thetas [n_rec], target [B*R, n_rec] complex128 and a dict of
    solver options: restart, tol, maxit; circulant (True or False: tables with or
    without the circulant form) and sstep (Newton vectors per block of s-step
    solves, 0 for one-vector ones), both chosen by the sizes when absent or
    None."""

    @staticmethod
    def forward(ctx, centers, radii, k, n_modes, disk_off, betas, thetas, target, opts=None):
        opts = dict(opts or {})
        c = centers.detach().cpu().numpy()
        a = radii.detach().cpu().numpy()
        kk = k.detach().cpu().numpy().reshape(-1)
        nm = np.asarray(n_modes)
        off = np.asarray(disk_off)
        inst = [(c[off[b]:off[b + 1]], a[off[b]:off[b + 1]], nm[off[b]:off[b + 1]], kk[b])
                for b in range(len(off) - 1)]
        dev = centers.device if centers.is_cuda else torch.device("cuda")
        loss, dc, da, dk = _misfit_grad(inst, str(dev), betas, thetas, target, opts)
        inst_of = torch.as_tensor(np.repeat(np.arange(len(off) - 1), np.diff(off)), device=dc.device)
        ctx.save_for_backward(dc, da, dk, inst_of)
        return loss.to(centers.device)

    @staticmethod
    def backward(ctx, gl):
        dc, da, dk, inst_of = ctx.saved_tensors
        g = gl.to(dc.device)
        gi = g[inst_of]
        return (dc * gi[:, None]).to(gl.device), (da * gi).to(gl.device), (dk * g).to(gl.device), \
            None, None, None, None, None, None
