"""Near field against the oracle on both sides of each switch of its Hankel
functions (k r at 0.05, 5, 12, 25, 50 and 100), for 1 to 5 right-hand sides (1, 2
and 4 per thread, with a remainder), and with the coefficients of 1 to 16 disks
staged at a time.  Each point's error is against the sum of the magnitudes of its
terms: N_p eps from the recurrence over orders and k r eps <= 200 eps from the phase,
1e-12 with a margin of ten."""
import numpy as np
import pytest
import torch

import synth
from oracle import nearfield
from oracle.bessel import besselj, hankel1

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,ka,R", [
    (1, 0, 1e-3, 1), (1, 2, 1e-3, 2), (1, 9, 2.0, 3), (16, 3, 0.5, 4), (17, 2, 0.04, 1), (33, 5, 0.3, 5),
    (35, 12, 4.0, 2), (5, 40, 20.0, 4), (3, 200, 150.0, 1), (2, 200, 110.0, 3)])
def test_ranges(M, N, ka, R):
    from paper_1409_8186_amd import Problem
    k = 2.0
    rng = np.random.default_rng(M + N)
    side = int(np.ceil(np.sqrt(M)))
    cen = 2.5 * ka / k * np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:M]
    orders = rng.integers(max(0, N - 2), N + 1, M).astype(np.int32)
    orders[-1] = N
    cl = synth.Cluster(cen, np.full(M, ka / k), orders, k)
    x = np.array([1.001 * ka, 0.01, 0.04999, 0.05001, 1.0, 4.999, 5.001, 8.0, 11.99, 12.01, 20.0, 24.99, 25.01,
                  40.0, 49.9, 50.1, 80.0, 99.9, 100.1, 170.0, 0.5 * ka])
    t = rng.uniform(0.0, 2.0 * np.pi, (13, len(x)))
    pts = (x / k)[None, :, None] * np.stack([np.cos(t), np.sin(t)], -1)
    pts = pts.reshape(-1, 2)                               # 273 points: a full workgroup and a part
    n = int(np.sum(2 * orders + 1))
    rho = rng.normal(size=(R, n)) + 1j * rng.normal(size=(R, n))
    # the H_m grow like (m / (e k a))^m: densities that make the orders' terms alike on the circle
    m = np.concatenate([np.arange(-q, q + 1) for q in orders])
    rho /= np.abs(besselj(m, ka) * hankel1(m, ka))[None, :]
    u = Problem.from_cluster(cl).nearfield(torch.tensor(rho.reshape(-1), device="cuda"), pts, R=R).cpu().numpy()
    ref = nearfield.potential(cl.centers, cl.radii, cl.n_modes, k, rho, pts)
    size = np.zeros((R, len(pts)))
    off = 0
    for p in range(M):
        q = np.arange(-orders[p], orders[p] + 1)
        r = np.hypot(*(pts - cl.centers[p]).T)
        h = np.abs(hankel1(q[None, :], k * np.maximum(r, cl.radii[p])[:, None]))
        c = np.abs(rho[:, off:off + len(q)] * besselj(q, ka)) * np.sqrt(np.pi * cl.radii[p] / 8)
        size += c @ h.T
        off += len(q)
    # a point on a circle to rounding (k r = k a = 20) is inside or not as the distance rounds
    gap = np.min(np.abs(np.hypot(*(pts[:, None] - cl.centers[None]).transpose(2, 0, 1)) / cl.radii - 1.0), 1)
    ok = gap > 1e-12
    assert np.array_equal(u[:, ok] == 0.0, ref[:, ok] == 0.0)
    u, ref, size = u[:, ok], ref[:, ok], size[:, ok]
    err = np.max(np.abs(u - ref) / size)
    print(M, N, ka, R, "err %.2e" % err, flush=True)
    assert err < 1e-12


@pytest.mark.parametrize("M,R", [(2, 1), (9, 3), (40, 2)])
def test_few_points_as_many(M, R):
    """The same points alone (disks split over the waves) and among 300,000 (not split)."""
    from paper_1409_8186_amd import Problem
    rng = np.random.default_rng(M)
    side = int(np.ceil(np.sqrt(M)))
    cen = 3.0 * np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:M]
    cl = synth.Cluster(cen, np.full(M, 0.8), rng.integers(3, 12, M).astype(np.int32), 5.0)
    pr = Problem.from_cluster(cl)
    rho = torch.tensor(rng.normal(size=R * cl.n_tot) + 1j * rng.normal(size=R * cl.n_tot), device="cuda")
    pts = rng.uniform(-2.0, 3.0 * side, (300000, 2))
    pick = np.sort(rng.choice(len(pts), 333, replace=False))
    many = pr.nearfield(rho, pts, R=R).cpu().numpy()[:, pick]
    few = pr.nearfield(rho, pts[pick], R=R).cpu().numpy()
    assert np.array_equal(many == 0.0, few == 0.0)
    # sums of the same terms in another order: eps times the terms, some of which cancel
    assert np.max(np.abs(many - few)) < 1e-12 * np.max(np.abs(many))
