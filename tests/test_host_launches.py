"""Launch shapes and routes on the host alone (tests/native/build_host.py: kernels are recorded,
not run, so their buffers need not exist)."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "native"))
import build_host  # noqa: E402

GRID_THREADS = 2 ** 32  # a launch has fewer threads along x


@pytest.fixture(scope="module")
def host():
    return build_host.Host()


def line(M, N, k=5.0):
    return np.stack([4.0 * np.arange(M), np.zeros(M)], 1), np.ones(M), np.full(M, N), k


@pytest.mark.parametrize("M,R,n_theta", [(8, 1024, 1 << 20), (3, 1024, 1 << 20), (70, 4096, 300000), (8, 16, 67108000),
                                         (8, 300, 20000), (3, 40, 1 << 20)])
def test_farfield_grid_within_the_launch_limit(host, M, R, n_theta):
    h = host.tables([line(M, 5)])
    host.launches.clear()
    host.check(host.lib.mudiff_farfield(h, R, 256, n_theta, 256, 256, None))
    (name, (gx, gy, _), threads, _, _), = host.launches
    assert gx * threads < GRID_THREADS and gy <= 65535, (name, gx, threads)
    host.check(host.lib.mudiff_destroy(h))
