"""Far field of many columns (matrix cores) against the oracle at the edges of its
tiles: 16 columns, 16 angles, 4 modes a step, 16 waves of one or four disks; with a
set operator's complex factors; and just below its limits, where the other kernel
runs.  Tolerance 1e-13 as for the far field elsewhere, times the size of the phases
k |O_p| <= 200 over 10 (the phase of e^{-i k theta . O_p} rounds by eps k |O_p|)."""
import numpy as np
import pytest
import torch

import synth
from oracle import farfield

pytestmark = pytest.mark.gpu


def _cluster(M, orders, seed, k):
    rng = np.random.default_rng(seed)
    side = int(np.ceil(np.sqrt(M)))
    c = 2.0 * np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:M]
    return synth.Cluster(c + rng.uniform(-0.3, 0.3, (M, 2)), rng.uniform(0.3, 0.6, M),
                         rng.choice(np.asarray(orders, np.int32), M).astype(np.int32), k)


@pytest.mark.parametrize("M,orders,R,n_theta", [
    (1, [0], 4, 1), (4, [1, 2], 5, 17), (5, [3], 16, 16), (17, [2, 5], 17, 33), (63, [1, 7], 4, 15),
    (64, [4, 9], 33, 250), (65, [6, 31], 16, 520), (70, [0, 40], 32, 257), (70, [5], 3, 40), (66, [5], 8, 40)])
def test_matches_oracle(M, orders, R, n_theta):
    from paper_1409_8186_amd import Problem
    cls = [_cluster(M, orders, 1, 6.0), _cluster(max(1, M - 3), orders, 2, 5.0)]
    pr = Problem.from_clusters(cls)
    rng = np.random.default_rng(3)
    th = np.sort(rng.uniform(0.0, 2.0 * np.pi, n_theta))
    X = [rng.normal(size=(R, int(n))) + 1j * rng.normal(size=(R, int(n))) for n in pr.n_tot]
    a = pr.farfield(pr.pack(X), th, R=R).cpu().numpy()
    for b, c in enumerate(cls):
        ref = np.stack([farfield.farfield(c.centers, c.radii, c.n_modes, c.k, th, x) for x in X[b]])
        err = np.linalg.norm(a[b * R:(b + 1) * R] - ref) / np.linalg.norm(ref)
        print(M, R, n_theta, "instance", b, "err %.2e" % err, flush=True)
        assert err < 2e-12


def test_set_operator():
    """Brakhage-Werner far field (complex factors): 16 columns at once against one by one."""
    from paper_1409_8186_amd import Problem
    c = _cluster(20, [3, 6], 4, 4.0)
    pr = Problem.from_cluster(c)
    pr.set_operator("bwie")
    rng = np.random.default_rng(5)
    x = torch.tensor(rng.normal(size=(16, c.n_tot)) + 1j * rng.normal(size=(16, c.n_tot)), device="cuda")
    th = np.linspace(0.0, 6.0, 50)
    a = pr.farfield(x.reshape(-1), th, R=16)
    for r in (0, 7, 15):
        one = pr.farfield(x[r].contiguous(), th, R=1)[0]
        assert float((a[r] - one).norm()) < 2e-12 * float(one.norm())
