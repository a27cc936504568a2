"""Uniform orders, one lane per pair, one row disk or (from 400 waves, 135 disks, on) four
per workgroup: against the oracle's
dense matrix at row counts with every remainder of four and chunks of 64 column disks
whose last has 1, 2, 7, 8, 11, 12, 13 and 64 of them; several instances, columns and a
set operator's complex column factors.  1e-12 as for the applies elsewhere."""
import numpy as np
import pytest
import torch

import synth
from oracle import operator

pytestmark = pytest.mark.gpu


def _cluster(M, N, seed):
    rng = np.random.default_rng(seed)
    side = int(np.ceil(np.sqrt(M)))
    c = 2.0 * np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:M]
    return synth.Cluster(c + rng.uniform(-0.3, 0.3, (M, 2)), np.full(M, 0.5), np.full(M, N, np.int32),
                         max(0.5, N / 2.0))


@pytest.mark.parametrize("Ms,N,R", [([65], 1, 1), ([66], 3, 2), ([67], 12, 1), ([72, 17], 12, 3), ([73], 7, 1),
                                    ([76], 5, 7), ([77], 12, 1), ([78, 1, 20], 2, 2), ([129], 4, 1), ([130], 4, 1), ([135], 1, 2),
                                    ([136], 4, 1), ([137], 12, 1), ([140], 2, 7), ([141], 6, 2), ([142], 3, 1),
                                    ([100, 101, 103, 66], 5, 3)])
def test_matches_dense(Ms, N, R):
    from paper_1409_8186_amd import Problem
    cls = [_cluster(M, N, M) for M in Ms]
    pr = Problem.from_clusters(cls)
    assert pr.apply_config(R)["kind"] == "lane"
    rng = np.random.default_rng(R)
    X = [rng.normal(size=(R, c.n_tot)) + 1j * rng.normal(size=(R, c.n_tot)) for c in cls]
    for op in (0, 1):
        for c, x, v in zip(cls, X, pr.split(pr.matvec(pr.pack(X), R=R, op=op), R)):
            L = operator.efie_matrix(c.centers, c.radii, c.n_modes, c.k)
            ref = x @ (L / np.diag(L)[:, None] if op else L).T
            err = np.linalg.norm(v.cpu().numpy() - ref) / np.linalg.norm(ref)
            print(Ms, N, R, op, "err %.2e" % err, flush=True)
            assert err < 1e-12


def test_operator():
    """Against the matrix-core apply of eight columns."""
    from paper_1409_8186_amd import Problem
    c = _cluster(138, 6, 1)
    pr = Problem.from_cluster(c)
    pr.set_operator("bwie")
    rng = np.random.default_rng(0)
    x = torch.tensor(rng.normal(size=(8, c.n_tot)) + 1j * rng.normal(size=(8, c.n_tot)), device="cuda")
    ref = pr.matvec(x.reshape(-1), R=8).reshape(8, -1)[:2]
    got = pr.matvec(x[:2].reshape(-1).contiguous(), R=2).reshape(2, -1)
    assert float((got - ref).norm() / ref.norm()) < 1e-12
