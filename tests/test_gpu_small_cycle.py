"""GMRES cycles of small columns in one workgroup against the oracle's dense solve: rows
of one disk on both sides of a task's 32 outputs, orders 0 to 200, up to the largest
instance taken (16 disks, 512 rows) and just beyond, basis in LDS and in global memory,
cycles that end inside and by their length, several instances, columns and operators.
Solved to 1e-12; the matrices' condition numbers are below 1e3: 1e-9."""
import numpy as np
import pytest
import torch

import synth
from oracle import operator, rhs, solve

pytestmark = pytest.mark.gpu


def _cluster(orders, seed, k=1.0):
    rng = np.random.default_rng(seed)
    N = np.asarray(orders, np.int32)
    a = np.maximum(0.3, (N - 6.0) * 0.6) / k
    pitch = 2.4 * a.max() + 0.5
    side = int(np.ceil(np.sqrt(len(N))))
    c = pitch * np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:len(N)]
    return synth.Cluster(c + rng.uniform(-0.05, 0.05, (len(N), 2)) * pitch, a, N, k)


@pytest.mark.parametrize("orders,R,restart,graph", [
    ([[0]], 1, 5, False), ([[3]], 2, 30, False), ([[200]], 1, 12, False), ([[0, 0]], 3, 4, False),
    ([[15, 16, 3]], 7, 30, False), ([[15] * 4], 1, 5, True), ([[4, 9, 0, 31, 32]], 2, 50, False),
    ([[127, 127]], 1, 20, False), ([[7] * 16], 1, 30, False), ([[7] * 17], 1, 30, False),
    ([[12] * 10, [5, 9], [16] * 4, [1]], 5, 15, True), ([[16, 18, 20, 15, 17, 19, 16, 20, 15, 18, 17]], 2, 64, False)])
def test_matches_dense_solve(orders, R, restart, graph):
    from paper_1409_8186_amd import Problem
    cls = [_cluster(o, i, 1.0 + 0.1 * i) for i, o in enumerate(orders)]
    pr = Problem.from_clusters(cls)
    betas = np.stack([synth.uniform_angles(R) + 0.3 * i for i in range(len(cls))])
    rho, flag, _, iters, _ = pr.gmres(betas=betas, restart=restart, tol=1e-12, maxit=4000, graph=graph)
    assert torch.all(flag == 0), flag
    print(orders, R, restart, "iterations", int(iters.max()), flush=True)
    for b, (c, y) in enumerate(zip(cls, pr.split(rho, R))):
        L = operator.efie_matrix(c.centers, c.radii, c.n_modes, c.k)
        ref = solve.efie_solve_lu(L, rhs.planewave(c.centers, c.radii, c.n_modes, c.k, betas[b]))
        # per mode in the preconditioned scaling: rho's entries span the range of 1 / (J_m H_m)
        d = np.abs(np.diag(L))[None, :]
        assert np.linalg.norm((y.cpu().numpy() - ref) * d) < 1e-9 * np.linalg.norm(ref * d)


@pytest.mark.parametrize("name", ["mfie", "cfie", "bwie"])
def test_operators(name):
    """The same system solved with another number of columns (matrix-core apply)."""
    from paper_1409_8186_amd import Problem
    pr = Problem.from_cluster(_cluster([5, 8, 6, 9], 3))
    pr.set_operator(name)
    b8 = np.linspace(0.0, 6.0, 8)[None]
    ref = pr.gmres(betas=b8, restart=25, tol=1e-12)[0]
    got, flag = pr.gmres(betas=b8[:, :3], restart=25, tol=1e-12)[:2]
    assert torch.all(flag == 0)
    ref = ref.reshape(8, -1)[:3]
    assert float((got.reshape(3, -1) - ref).norm() / ref.norm()) < 1e-9
