"""Batches with instances inside and outside the circulant form: the queue of the latter runs on a
second stream in eager applies and on the caller's in a captured one.  Eager applies and replays of
a caller's graph against the direct form, on changing inputs; 1e-12 as for the circulant form
elsewhere."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


def _cluster(rng, M, pitch):
    side = int(np.ceil(np.sqrt(M)))
    c = pitch * np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:M].astype(float)
    return synth.Cluster(c + rng.uniform(-0.02, 0.02, (M, 2)), rng.uniform(0.8, 0.95, M),
                         rng.integers(16, 24, M).astype(np.int32), 5.0)


@pytest.mark.parametrize("M,m,R", [(150, 10, 8), (120, 7, 33)])
def test_queue_in_eager_and_captured_applies(M, m, R):
    from paper_1409_8186_amd import Problem
    rng = np.random.default_rng(M + R)
    pr = Problem.from_clusters([_cluster(rng, M, 10.0), _cluster(rng, m, 2.1)], circulant=True)
    n = R * int(pr.n_tot.sum())
    xs = [torch.tensor(rng.normal(size=n) + 1j * rng.normal(size=n), device="cuda") for _ in range(4)]
    pr.set_circulant(R, 0)
    ref = [pr.matvec(x, R=R) for x in xs]
    pr.set_circulant(R, 1)

    def close(y, r):
        return float((y - r).norm() / r.norm()) < 1e-12

    for x, r in zip(xs, ref):
        assert close(pr.matvec(x, R=R), r)
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
    # the tile that was timed, fixed, and the form switched off: the direct form again
    pr.set_circulant_tile(R, *pr.circulant_tile(R))
    assert close(pr.matvec(xs[2], R=R), ref[2])
    pr.set_circulant(R, 0)
    assert close(pr.matvec(xs[3], R=R), ref[3])
