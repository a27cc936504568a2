"""Close pairs on a second stream beside the transforms and products (medium sizes of
the circulant form): back-to-back applies on changing inputs, replays of a caller's
graph (where everything stays on one stream) and a solve replayed as graphs, against
the direct form; below the rule's range too.  1e-12 as for the circulant form elsewhere."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,R", [(120, 64), (250, 32), (400, 8), (30, 16)])
def test_beside(M, R):
    from paper_1409_8186_amd import Problem
    rng = np.random.default_rng(M)
    side = int(np.ceil(np.sqrt(M)))
    c = 2.6 * np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:M]
    cl = synth.Cluster(c + rng.uniform(-0.2, 0.2, (M, 2)), rng.uniform(0.4, 0.9, M),
                       rng.integers(9, 14, M).astype(np.int32), 6.0)
    pr = Problem.from_clusters([cl], circulant=True)
    n = R * cl.n_tot
    xs = [torch.tensor(rng.normal(size=n) + 1j * rng.normal(size=n), device="cuda") for _ in range(4)]
    pr.set_circulant(R, 0)
    ref = [pr.matvec(x, R=R) for x in xs]
    pr.set_circulant(R, 1)

    def close(y, r):
        return float((y - r).norm() / r.norm()) < 1e-12

    for x, r in zip(xs, ref):
        pr.matvec(x, R=R)
        y = pr.matvec(pr.matvec(x, R=R) * 0 + x, R=R)  # an input freed at once
        assert close(y, r)
    assert pr.apply_config(R)["kind"] == "circulant"
    x, y = xs[0].clone(), torch.empty_like(xs[0])
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        pr.matvec(x, R=R, out=y)
    for k in (1, 2, 3):
        x.copy_(xs[k])
        assert close(pr.matvec(xs[k - 1], R=R), ref[k - 1])
        g.replay()
        torch.cuda.synchronize()
        assert close(y, ref[k]), k
    betas = np.linspace(0.0, 6.0, R)[None]
    a = pr.gmres(betas=betas, restart=20, tol=1e-10, graph=True)[0]
    b = pr.gmres(betas=betas, restart=20, tol=1e-10, graph=False)[0]
    assert float((a - b).norm() / b.norm()) < 1e-8  # two solves to 1e-10
