"""Which tables and solver the misfit function takes: by rule, as the caller asks, and what is left
where they fail (no room for the circulant tables, an s-step solve that stagnates).  On the CPU with
a stand-in for Problem; on the device the gradient of each form against the oracle's."""
import numpy as np
import pytest
import torch

import synth
from paper_1409_8186_amd import _lib as L
from paper_1409_8186_amd import autograd


class Fake:
    """Problem that fails as `fails` says for (circulant, s-step vectors), and notes its uses."""
    fails, calls, open = {}, [], 0

    def __init__(self, inst, device, circulant):
        assert not Fake.open  # the one that failed is closed first
        if Fake.fails.get((circulant, "tables")):
            Fake.calls.append((circulant, "tables"))
            raise torch.OutOfMemoryError("tables")
        self.circulant, self.M, self.B = circulant, sum(len(i[1]) for i in inst), len(inst)
        Fake.open += 1

    def grad(self, betas, thetas, target, restart, tol, maxit, flags):
        s = flags >> 16 & 255
        assert bool(flags & L.SSTEP) == (s > 0)
        Fake.calls.append((self.circulant, s))
        e = Fake.fails.get((self.circulant, s))
        if e:
            raise e
        z = torch.zeros(self.M, dtype=torch.float64)
        return torch.ones(self.B, dtype=torch.float64), torch.zeros(self.M, 2, dtype=torch.float64), z, z[:self.B]

    def close(self):
        Fake.open -= 1


OOM = torch.OutOfMemoryError("workspace")
STUCK = L.MudiffError(5, "forward solve did not converge")


def run(monkeypatch, B, M, N, R, opts, fails):
    """(calls, what was raised) of a gradient of B instances of M disks of order N."""
    monkeypatch.setattr(autograd, "Problem", Fake)
    Fake.fails, Fake.calls, Fake.open = fails, [], 0
    c = torch.zeros(B * M, 2, dtype=torch.float64, requires_grad=True)
    args = (c, torch.ones(B * M, dtype=torch.float64), torch.ones(B, dtype=torch.float64), np.full(B * M, N),
            np.arange(B + 1) * M, np.zeros((B, R)), np.zeros(3), np.zeros((B * R, 3), complex), opts)
    err = None
    try:
        autograd.FarFieldMisfit.apply(*args).sum().backward()
        assert c.grad.shape == (B * M, 2)
    except (torch.OutOfMemoryError, L.MudiffError) as e:
        err = e
    assert Fake.open == 0
    return Fake.calls, err


@pytest.mark.parametrize("B,M,N,R,opts,call", [
    (2, 60, 4, 7, {}, (False, 0)), (2, 60, 4, 8, {}, (True, 10)), (2, 60, 32, 8, {}, (False, 0)),
    (2, 60, 4, 8, {"restart": 65}, (True, 0)), (2, 60, 4, 8, {"restart": 19}, (True, 0)),
    (1, 30, 4, 8, {}, (True, 0)), (4, 30, 31, 8, {}, (True, 10)),
    (16, 10, 31, 64, {}, (True, 0)), (4, 10, 16, 64, {}, (False, 0)), (200, 3, 4, 64, {}, (False, 0)),
    (32, 16, 31, 64, {}, (True, 0)), (1, 2, 4, 8, {}, (False, 0)),
    (2, 60, 4, 8, {"circulant": False, "sstep": 0}, (False, 0)),
    (2, 2, 4, 2, {"circulant": True, "sstep": 4}, (True, 4)),
    (2, 60, 4, 8, {"circulant": None, "sstep": None}, (True, 10)),
])
def test_form_and_solver(monkeypatch, B, M, N, R, opts, call):
    assert run(monkeypatch, B, M, N, R, opts, {}) == ([call], None)


@pytest.mark.parametrize("opts,fails,calls", [
    ({}, {(True, "tables"): True}, [(True, "tables"), (False, 0)]),
    ({}, {(True, 10): OOM}, [(True, 10), (False, 0)]),
    ({"sstep": 5}, {(True, 5): OOM}, [(True, 5), (False, 5)]),
    ({}, {(True, 10): STUCK}, [(True, 10), (True, 0)]),
    ({}, {(True, 10): STUCK, (True, 0): OOM}, [(True, 10), (True, 0), (False, 0)]),
    # what nothing is left for is raised, and so is what the caller asked for
    ({"circulant": False, "sstep": 0}, {(False, 0): OOM}, [(False, 0)]),
    ({"circulant": False, "sstep": 0}, {(False, 0): STUCK}, [(False, 0)]),
    ({}, {(True, 10): STUCK, (True, 0): STUCK}, [(True, 10), (True, 0)]),
    ({}, {(True, 10): L.MudiffError(4, "device")}, [(True, 10)]),
    ({"circulant": True, "sstep": 6}, {(True, 6): STUCK}, [(True, 6)]),
    ({"circulant": True, "sstep": 0}, {(True, 0): OOM}, [(True, 0)]),
])
def test_what_is_left_after_a_failure(monkeypatch, opts, fails, calls):
    got, err = run(monkeypatch, 2, 60, 4, 8, opts, fails)
    assert got == calls
    last = fails.get(calls[-1])
    assert err is None if last is None else type(err) is type(last)


@pytest.mark.gpu
@pytest.mark.parametrize("opts", [{}, {"circulant": True, "sstep": 10}, {"circulant": False, "sstep": 10}, {"circulant": True}])
def test_gradient_of_many_columns(opts):
    """8 and 17 incidences on two instances of well-separated disks: the oracle's adjoint gradient to
    1e-10, as for the direct form and one-vector solves."""
    from oracle import gradient
    from paper_1409_8186_amd import FarFieldMisfit
    for R, M in ((8, 9), (17, 6)):
        cls, targets = [], []
        for i in range(2):
            base = synth.small_random(80 + i, M, 0.4, 0.7, 30.0, 2.0, 3.0, 4, R=R, n_theta=6)
            tgt = synth.perturb(np.random.default_rng(180 + i), base)
            cls.append(base)
            targets.append(gradient.forward(tgt.centers, tgt.radii, tgt.n_modes, tgt.k, base.betas, base.thetas))
        leaf = [torch.tensor(v, dtype=torch.float64, device="cuda", requires_grad=True) for v in
                (np.concatenate([c.centers for c in cls]), np.concatenate([c.radii for c in cls]), [c.k for c in cls])]
        loss = FarFieldMisfit.apply(*leaf, np.concatenate([c.n_modes for c in cls]), np.array([0, M, 2 * M]),
                                    np.stack([c.betas for c in cls]), cls[0].thetas, np.concatenate(targets),
                                    {"tol": 1e-13, **opts})
        loss.sum().backward()
        dc, da, dk = (v.grad.cpu().numpy() for v in leaf)
        for b, (c, t) in enumerate(zip(cls, targets)):
            l0, dc0, da0, dk0 = gradient.misfit_grad(c.centers, c.radii, c.n_modes, c.k, c.betas, c.thetas, t)
            g = np.concatenate([dc[b * M:(b + 1) * M].ravel(), da[b * M:(b + 1) * M], [dk[b]]])
            g0 = np.concatenate([dc0.ravel(), da0, [dk0]])
            assert abs(loss[b].item() - l0) <= 1e-10 * l0
            assert np.linalg.norm(g - g0) < 1e-10 * np.linalg.norm(g0), (R, b, opts)
