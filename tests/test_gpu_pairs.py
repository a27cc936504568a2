"""The one-lane-per-pair apply for differing orders (few right-hand sides) at the
edges of its tiles: blocks of 1 to 14 outputs (n_p = 1 .. 63), chunks of 64
column disks (24, 64, 65, 129 disks), both block widths, segments of several
chunks, and the batches that stay with the LDS-staged kernel.

Tolerance 1e-12, normwise per column: the apply sums N_tot products of O(1)
terms; the symbols' recurrences of up to 62 steps add at most about 62 * 4 eps
= 6e-14 relative to |H_nu|."""
import numpy as np
import pytest
import torch

import synth
from oracle import operator

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    from paper_1409_8186_amd import Problem
    assert torch.cuda.is_available()
    return Problem


def _grid(M, orders, seed, k=6.0, spacing=1.6):
    """M disks of radius 0.3..0.5 on a jittered grid, orders drawn from `orders`."""
    rng = np.random.default_rng(seed)
    side = int(np.ceil(np.sqrt(M)))
    g = spacing * np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:M]
    c = g + rng.uniform(-0.2, 0.2, (M, 2))
    return synth.Cluster(c, rng.uniform(0.3, 0.5, M), rng.choice(np.asarray(orders, np.int32), M).astype(np.int32), k)


def _vec(R, n, seed):
    rng = np.random.default_rng(seed)
    return rng.normal(size=(R, n)) + 1j * rng.normal(size=(R, n))


CASES = {
    "orders 0..31, 24 disks": lambda: [_grid(24, range(32), 1)],
    "64 disks": lambda: [_grid(64, [2, 5, 9], 2)],
    "65 disks": lambda: [_grid(65, [6, 7, 13], 3)],
    "129 disks, wide blocks in the batch": lambda: [_grid(129, [3, 10, 17], 4), _grid(30, [0, 1], 5)] +
    [_grid(100, [14, 16, 19], 20 + i) for i in range(12)],
    "one order above the lane kernel's": lambda: [_grid(26, [15], 6)],
    "an order above 31": lambda: [_grid(25, [4, 32], 7)],
    "few disks": lambda: [_grid(23, [3, 8], 8), synth.Cluster(np.zeros((1, 2)), np.ones(1), np.array([5]), 2.0)],
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("R", [1, 7])
def test_apply_matches_oracle(P, name, R):
    cls = CASES[name]()
    pr = P.from_clusters(cls)
    assert pr.apply_config(R)["kind"] == "generic"
    X = [_vec(R, int(n), 100 + i) for i, n in enumerate(pr.n_tot)]
    x = pr.pack(X)
    mats = [operator.efie_matrix(c.centers, c.radii, c.n_modes, c.k) for c in cls]
    for op in (0, 1, 2):
        y = pr.split(pr.matvec(x, R=R, op=op), R)
        for i, (L, c) in enumerate(zip(mats, cls)):
            D = np.diag(L)
            ref = X[i] @ L.T if op == 0 else (X[i] @ L.T / D if op == 1 else X[i] @ L)
            got = y[i].cpu().numpy()
            err = np.max(np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1))
            print(name, "R", R, "op", op, "instance", i, "err %.2e" % err, flush=True)
            assert err < 1e-12


def test_segments_of_several_chunks(P):
    """2,944 disks of orders 0 and 1: the partial sums of one chunk each would
    exceed the scratch bound, so an item walks several chunks."""
    cl = _grid(2944, [0, 1], 9, k=1.0)
    pr = P.from_cluster(cl)
    X = _vec(2, cl.n_tot, 11)
    y = pr.matvec(torch.tensor(X.ravel(), device="cuda"), R=2, op=0).cpu().numpy().reshape(2, -1)
    off = np.concatenate([[0], np.cumsum(2 * cl.n_modes + 1)])
    for p in (0, 63, 64, 1500, 2943):
        ref = X @ operator.efie_row_block(cl.centers, cl.radii, cl.n_modes, cl.k, p).T
        got = y[:, off[p]:off[p + 1]]
        err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        print("row disk", p, "err %.2e" % err, flush=True)
        assert err < 1e-12


def test_set_operator_and_solve(P):
    """Complex column factors (CFIE) against the matrix-core path of the same
    handle, and GMRES, whose Gram-Schmidt kernel adds the chunk sums itself,
    against LU."""
    cl = _grid(70, [5, 8, 11], 12, k=4.0)
    pr = P.from_cluster(cl)
    rho, flag, *_ = pr.gmres(betas=[[0.3, 1.1]], tol=1e-12)
    L = operator.efie_matrix(cl.centers, cl.radii, cl.n_modes, cl.k)
    U = pr.rhs([[0.3, 1.1]]).cpu().numpy().reshape(2, -1)
    ref = np.linalg.solve(L, -U.T).T
    assert int(flag.abs().max()) == 0
    assert np.linalg.norm(rho.cpu().numpy().reshape(2, -1) - ref) < 1e-10 * np.linalg.norm(ref)
    pr.set_operator("cfie")
    X = _vec(8, cl.n_tot, 13)
    y8 = pr.matvec(torch.tensor(X.ravel(), device="cuda"), R=8, op=0).cpu().numpy().reshape(8, -1)
    y1 = pr.matvec(torch.tensor(X[:3].ravel(), device="cuda"), R=3, op=0).cpu().numpy().reshape(3, -1)
    assert np.linalg.norm(y1 - y8[:3]) < 1e-12 * np.linalg.norm(y8[:3])


def test_orders_beyond_the_pair_stay_finite(P):
    """Pairs so close (k b = 3e-4) that H_nu overflows at orders that other pairs
    of the instance need: such a batch stays with the LDS-staged kernel."""
    cl = _grid(24, [1, 2], 14, k=2e-4)
    cl.n_modes[3] = 31
    pr = P.from_cluster(cl)
    X = _vec(1, cl.n_tot, 15)
    y = pr.matvec(torch.tensor(X.ravel(), device="cuda"), R=1, op=1).cpu().numpy()
    assert np.isfinite(y).all()
    p = 5
    off = np.concatenate([[0], np.cumsum(2 * cl.n_modes + 1)])
    blk = operator.efie_row_block(cl.centers, cl.radii, cl.n_modes, cl.k, p)
    n = 2 * int(cl.n_modes[p]) + 1
    D = blk[np.arange(n), off[p] + np.arange(n)]
    ref = blk @ X[0] / D
    err = np.linalg.norm(y[off[p]:off[p + 1]] - ref) / np.linalg.norm(ref)
    print("row disk", p, "err %.2e" % err, flush=True)
    assert err < 1e-12
