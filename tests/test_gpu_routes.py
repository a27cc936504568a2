"""Kernels on either side of the rules that choose between them: applies against the oracle's dense
matrix (1e-12, as for the applies elsewhere) and solves against its LU factorisation."""
import numpy as np
import pytest
import torch

import synth
from oracle import operator, rhs, solve

pytestmark = pytest.mark.gpu


def cluster(M, orders, seed):
    rng = np.random.default_rng(seed)
    side = int(np.ceil(np.sqrt(M)))
    c = 2.0 * np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:M]
    n = rng.integers(orders[0], orders[1] + 1, M).astype(np.int32)
    return synth.Cluster(c + rng.uniform(-0.3, 0.3, (M, 2)), np.full(M, 0.5), n, max(0.5, orders[0] / 2.0))


def check_applies(cls, Rs, sample=None):
    from paper_1409_8186_amd import Problem
    pr = Problem.from_clusters(cls)
    rng = np.random.default_rng(len(cls))
    X = [rng.normal(size=(max(Rs), c.n_tot)) + 1j * rng.normal(size=(max(Rs), c.n_tot)) for c in cls]
    for R in Rs:
        for op in (0, 1):
            Y = pr.split(pr.matvec(pr.pack([x[:R] for x in X]), R=R, op=op), R)
            for b in (sample or range(len(cls))):
                c = cls[b]
                L = operator.efie_matrix(c.centers, c.radii, c.n_modes, c.k)
                ref = X[b][:R] @ (L / np.diag(L)[:, None] if op else L).T
                err = np.linalg.norm(Y[b].cpu().numpy() - ref) / np.linalg.norm(ref)
                print(b, R, op, "err %.2e" % err, flush=True)
                assert err < 1e-12


@pytest.mark.parametrize("Ms,N,R", [([134], 9, 1), ([135], 10, 2), ([136], 11, 1), ([137], 12, 3),
                                    ([100, 101, 103, 66], 9, 2)])
def test_four_rows_per_workgroup(Ms, N, R):
    check_applies([cluster(M, (N, N), M) for M in Ms], [R])


@pytest.mark.parametrize("B,M,N", [(1000, 4, 3), (300, 10, 2), (40, 12, 1)])
def test_uniform_orders_by_number_of_columns(B, M, N):
    """Whole rows per workgroup with one column, one lane per pair with seven."""
    check_applies([cluster(M, (N, N), b) for b in range(B)], [1, 7], sample=[0, B // 2, B - 1])


@pytest.mark.parametrize("Ms,orders", [([5, 12, 9, 7] * 25 + [24], (13, 20)), ([3] * 20 + [25], (24, 31)),
                                       ([26], (1, 4)), ([5, 12] * 20 + [70], (13, 20)), ([26], (13, 20)),
                                       ([17, 23], (15, 15)), ([65, 24], (15, 15)), ([66], (15, 15))])
def test_mixed_orders_by_the_whole_batch(Ms, orders):
    check_applies([cluster(M, orders, M + i) for i, M in enumerate(Ms)], [1, 4], sample=[0, len(Ms) - 1])


@pytest.mark.parametrize("B,M,orders,R", [(1, 11, (16, 16), 1), (1, 16, (12, 12), 2), (1, 12, (12, 12), 1),
                                          (1, 14, (5, 18), 1), (1, 8, (25, 25), 1), (270, 16, (12, 12), 7)])
def test_cycles_on_either_side(B, M, orders, R):
    """Three kernels a step, and whole cycles in one workgroup with the basis in LDS (12 disks of order
    12), in global memory (8 of order 25) and over several rounds of columns (270 x 16)."""
    from paper_1409_8186_amd import Problem
    cls = [cluster(M, orders, M + b) for b in range(B)]
    betas = np.linspace(0.3, 2.0, R)
    pr = Problem.from_clusters(cls)
    rho, flag, relres, _, _ = pr.gmres(betas=np.tile(betas, (B, 1)), restart=30, tol=1e-12, maxit=3000)
    assert int(flag.abs().max()) == 0 and float(relres.max()) <= 1e-12
    got = pr.split(rho, R)
    for b in {0, B // 2, B - 1}:
        c = cls[b]
        L = operator.efie_matrix(c.centers, c.radii, c.n_modes, c.k)
        ref = solve.efie_solve_lu(L, rhs.planewave(c.centers, c.radii, c.n_modes, c.k, betas))
        d = np.abs(np.diag(L))[None, :]  # in the preconditioned scaling
        e = np.linalg.norm((got[b].cpu().numpy() - ref) * d) / np.linalg.norm(ref * d)
        print(B, M, orders, R, b, "err %.2e" % e, flush=True)
        assert e < 1e-9  # a residual of 1e-12, condition below 1e3
