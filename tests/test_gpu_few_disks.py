"""Applies of few disks, whole rows per workgroup, against the oracle's dense matrix: rows
on both sides of a task's 32 outputs, orders 0 to 200, 1 to 16 disks (and 17, the next
kernel; uniform orders up to 12 on both sides of their rule), several instances and
columns, A, L and L^T, and set operators.
1e-12 as for the applies elsewhere."""
import numpy as np
import pytest
import torch

import synth
from oracle import operator

pytestmark = pytest.mark.gpu


def _cluster(orders, seed):
    rng = np.random.default_rng(seed)
    N = np.asarray(orders, np.int32)
    k = 1.0 + 0.2 * seed
    a = np.maximum(0.3, (N - 6.0) * 0.6) / k
    pitch = 2.4 * a.max() + 0.5
    side = int(np.ceil(np.sqrt(len(N))))
    c = pitch * np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:len(N)]
    return synth.Cluster(c + rng.uniform(-0.05, 0.05, (len(N), 2)) * pitch, a, N, k)


@pytest.mark.parametrize("orders,R", [
    ([[0]], 1), ([[40]], 2), ([[0, 0]], 3), ([[15, 16, 3]], 7), ([[15] * 4], 1), ([[4, 9, 0, 31, 32]], 2),
    ([[63, 64, 47]], 1), ([[200, 3]], 1), ([[7] * 16], 5), ([[7] * 17], 1), ([[14] * 16], 1), ([[5, 8] * 8], 2),
    ([[12] * 12, [12, 12], [12]], 3), ([[12] * 10, [5, 9], [16] * 4, [1], [33, 2, 8]], 5)])
def test_matches_dense(orders, R):
    from paper_1409_8186_amd import Problem
    cls = [_cluster(o, i) for i, o in enumerate(orders)]
    pr = Problem.from_clusters(cls)
    rng = np.random.default_rng(R)
    X = [rng.normal(size=(R, c.n_tot)) + 1j * rng.normal(size=(R, c.n_tot)) for c in cls]
    # entries in the scale of a solution's: the off-diagonal factors span J_m and 1 / H_m
    for op in (0, 1, 2):
        y = pr.split(pr.matvec(pr.pack(X), R=R, op=op), R)
        for c, x, v in zip(cls, X, y):
            L = operator.efie_matrix(c.centers, c.radii, c.n_modes, c.k)
            Mx = {0: L, 1: L / np.diag(L)[:, None], 2: L.T}[op]
            err = np.linalg.norm(v.cpu().numpy() - x @ Mx.T) / np.linalg.norm(x @ Mx.T)
            print(orders, R, op, "err %.2e" % err, flush=True)
            assert err < 1e-12


@pytest.mark.parametrize("name", ["mfie", "bwie", "neumann_sl"])
def test_operators(name):
    """Against the matrix-core apply of eight columns."""
    from paper_1409_8186_amd import Problem
    c = _cluster([5, 8, 20, 9, 17], 1)
    pr = Problem.from_cluster(c)
    pr.set_operator(name)
    rng = np.random.default_rng(0)
    x = torch.tensor(rng.normal(size=(8, c.n_tot)) + 1j * rng.normal(size=(8, c.n_tot)), device="cuda")
    for op in (0, 1):
        ref = pr.matvec(x.reshape(-1), R=8, op=op).reshape(8, -1)
        got = pr.matvec(x[:3].reshape(-1).contiguous(), R=3, op=op).reshape(3, -1)
        assert float((got - ref[:3]).norm() / ref[:3].norm()) < 1e-12
