"""Close pairs of the circulant form (one wave per row disk, column tile and pair of
row tiles) against the dense oracle at the edges of its schedule: rows with no
close pair, lists of 1, 8, 9 and 19 pairs (8 is the longest that one wave walks
alone), one to four row tiles, column tiles that fill a workgroup of four waves or
not, and an instance outside the form whose short work queue runs on the second
stream.  Tolerance 1e-12 as for every apply (sums of N_tot products of O(1) terms)."""
import numpy as np
import pytest
import torch

import synth
from oracle import operator

pytestmark = pytest.mark.gpu


def _clumps(sizes, order, seed, k):
    """Clumps of the given sizes, close inside (k b < 2 order) and far from each other."""
    rng = np.random.default_rng(seed)
    a = 0.35 * order / k / 5.0
    c = []
    for i, n in enumerate(sizes):
        w = int(np.ceil(np.sqrt(n)))
        g = np.stack(np.meshgrid(np.arange(w), np.arange(w)), -1).reshape(-1, 2)[:n] * (2.2 * a)
        c.append(g + np.array([60.0 * (i % 3), 60.0 * (i // 3)]))
    c = np.concatenate(c)
    n = rng.integers(max(0, order - 2), order + 1, len(c)).astype(np.int32)
    return synth.Cluster(c, np.full(len(c), a), n, k)


@pytest.mark.parametrize("order", [3, 12, 20, 29])
@pytest.mark.parametrize("R", [8, 9, 27])
def test_lists_and_tiles(order, R):
    from paper_1409_8186_amd import Problem
    sizes = [1, 2, 9, 10, 20, 1, 1]
    far = _clumps(sizes, order, order, 4.0)
    near = synth.small_random(5, 9, 0.3, 0.5, 6.0, 0.1, 1.0, 8)   # every pair close: direct
    pr = Problem.from_clusters([far, near], circulant=True)
    info = pr.circulant_info()
    assert info["near_pairs"] >= sum(n * (n - 1) for n in sizes) and info["far_pairs"] > 0
    pr.set_circulant(R, 1)
    pr.set_apply_config(R, 1, 8, 32, 512)
    rng = np.random.default_rng(R)
    X = [rng.normal(size=(R, int(n))) + 1j * rng.normal(size=(R, int(n))) for n in pr.n_tot]
    x = pr.pack(X)
    for rep in range(2):
        y = pr.split(pr.matvec(x, R=R, op=0), R)
        assert pr.apply_config(R)["kind"] == "circulant"
        for c, Xb, Y in zip((far, near), X, y):
            ref = Xb @ operator.efie_matrix(c.centers, c.radii, c.n_modes, c.k).T
            err = np.max(np.linalg.norm(Y.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1))
            print("order", order, "R", R, "M", c.M, "err %.2e" % err, flush=True)
            assert err < 1e-12


def test_schedules_of_several_column_counts_share_a_handle():
    """Alternating column counts and tiles on one handle: each keeps its schedule on
    the device, and those past the room for them are uploaded at every call."""
    from paper_1409_8186_amd import Problem
    cl = _clumps([1, 3, 10, 1], 9, 7, 4.0)
    pr = Problem.from_cluster(cl, circulant=True)
    L = operator.efie_matrix(cl.centers, cl.radii, cl.n_modes, cl.k)
    rng = np.random.default_rng(8)
    Rs = [8, 15, 8, 40, 15, 8] + list(range(8, 130, 3)) + [8, 40]
    for R in Rs:
        pr.set_circulant(R, R % 2)
        pr.set_apply_config(R, 1, 8, 0, 512)
        X = rng.normal(size=(R, cl.n_tot)) + 1j * rng.normal(size=(R, cl.n_tot))
        y = pr.matvec(torch.tensor(X.ravel(), device="cuda"), R=R, op=0).cpu().numpy().reshape(R, -1)
        ref = X @ L.T
        assert np.linalg.norm(y - ref) < 1e-12 * np.linalg.norm(ref), R
