"""Per-frequency products of the circulant form with every tile a caller may fix, at
disk counts on both sides of the tiles' edges (16 to 128 rows, K steps of 4 to 32 column
disks with one, two or three steps) and at column counts on both sides of the rules
(8, 9, 12, 17, 24, 48).  Oracle: the direct form on the same handle, 1e-12 as for the
circulant form elsewhere."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,R", [(17, 8), (15, 9), (33, 11), (81, 12), (16, 16), (65, 17), (40, 23), (80, 24),
                                 (97, 33), (31, 47), (49, 48), (64, 70)])
def test_tiles(M, R):
    from paper_1409_8186_amd import Problem
    rng = np.random.default_rng(10 * M + R)
    side = int(np.ceil(np.sqrt(M)))
    c = 6.0 * np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:M]
    cl = synth.Cluster(c + rng.uniform(-0.5, 0.5, (M, 2)), rng.uniform(0.3, 0.5, M),
                       rng.integers(4, 7, M).astype(np.int32), 5.0)
    pr = Problem.from_clusters([cl], circulant=True)
    x = torch.tensor(rng.normal(size=R * cl.n_tot) + 1j * rng.normal(size=R * cl.n_tot), device="cuda")
    pr.set_circulant(R, 0)
    ref = pr.matvec(x, R=R)
    pr.set_circulant(R, 1)
    for tile in [None] + pr.circulant_tiles(R):
        if tile:
            pr.set_circulant_tile(R, *tile)
        y = pr.matvec(x, R=R)
        assert pr.apply_config(R)["kind"] == "circulant"
        assert float((y - ref).norm() / ref.norm()) < 1e-12, tile
