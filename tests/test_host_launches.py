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


@pytest.mark.parametrize("B,M,N,n_theta,R,mfma", [
    # (us of the other kernel and of the matrix-core kernel)
    (64, 12, 2, 3600, 4, False), (64, 12, 2, 360, 4, False),  # 207, 265; 23.5, 30.0
    (64, 12, 2, 360, 6, True), (64, 12, 12, 360, 4, True),    # 34, 30; 44.8, 44.1
    (500, 6, 2, 3600, 4, False), (64, 3, 0, 3600, 4, True),   # 1327, 1690
    (1, 50, 2, 360, 16, False), (1, 63, 0, 36, 4, False),     # 10.9, 12.7
    (1, 50, 2, 3600, 5, True), (1, 50, 12, 360, 4, True),     # 24.6, 21.6
    (1, 16, 2, 1, 4, True), (1, 30, 2, 36, 4, True), (1, 8, 12, 36, 3, False),
    (1, 300, 5, 36, 8, False), (1, 100, 2, 3600, 8, True),
])
def test_farfield_kernel_of_few_columns(host, B, M, N, n_theta, R, mfma):
    h = host.tables([line(M, N)] * B)
    host.launches.clear()
    host.check(host.lib.mudiff_farfield(h, R, 256, n_theta, 256, 256, None))
    assert ("k_farfield_mfma" in host.launches[0][0]) == mfma
    host.check(host.lib.mudiff_destroy(h))


def batch(sizes, lo, hi):
    """Instances of the given numbers of disks, on grids, with orders lo..hi in turn."""
    out = []
    for M in sizes:
        w = int(np.ceil(np.sqrt(M)))
        c = np.array([(i % w, i // w) for i in range(M)], float) * 4.0
        out.append((c, np.ones(M), lo + np.arange(M) * 7 % (hi - lo + 1), 5.0))
    return out


SMALL, TINY = [5 + i % 8 for i in range(1000)], [2 + i % 3 for i in range(300)]


@pytest.mark.parametrize("sizes,orders,kernel", [
    # a large instance among small ones: by what the whole batch takes (us, LDS-staged and one lane
    # per pair, below)
    (SMALL[:100] + [24], (13, 20), "k_apply"),         # 24.5, 31.7
    (SMALL + [24], (13, 20), "k_apply"),               # 188, 235
    (SMALL + [24] * 5, (24, 31), "k_apply"),           # 307, 483
    (TINY + [24], (24, 31), "k_apply"),                # 38.9, 84
    (TINY + [24] * 5, (13, 20), "k_apply"),            # 26.9, 37.8
    (SMALL[:100] + [200], (13, 20), "k_apply_pairs"),  # 143, 52
    (SMALL + [24], (1, 4), "k_apply_pairs"),           # 97, 33
    # one size
    ([26], (1, 4), "k_apply"),                         # 7.9, 9.4
    ([28], (13, 20), "k_apply_pairs"),                 # 19.7, 14.6
    ([64] * 8, (13, 20), "k_apply_pairs"),             # 148, 27
    ([400], (13, 20), "k_apply_pairs"),
    ([40], (24, 31), "k_apply_pairs"),                 # 41, 20
    ([40], (24, 32), "k_apply"),                       # orders beyond the kernel's
    # one order that has a variant of its own
    ([24] * 40, (15, 15), "k_apply"), ([28] * 120, (15, 15), "k_apply"),  # 20.4, 25.2; 62.7, 77.2
    ([32] * 8, (15, 15), "k_apply"), ([65] * 40, (15, 15), "k_apply"),    # 9.9, 13.9; 94.9, 122.6
    ([50] * 120, (15, 15), "k_apply_pairs"),                              # 175, 148
    ([100], (15, 15), "k_apply_pairs"), ([24] * 120, (14, 14), "k_apply_pairs"),
])
def test_kernel_of_mixed_orders(host, sizes, orders, kernel):
    h = host.tables(batch(sizes, *orders))
    size = host.lib.mudiff_matvec_workspace_size(h, 1)
    host.launches.clear()
    host.check(host.lib.mudiff_matvec(h, 1, 256, 512, 1, 1024, size, None))
    assert kernel + "IL" in host.launches[0][0], host.launches[0][0]
    host.check(host.lib.mudiff_destroy(h))


def uniform(B, M, N):
    return batch([M] * B, N, N)


@pytest.mark.parametrize("B,M,N,R,few", [
    # (us of one lane per pair and of whole rows per workgroup)
    (1, 4, 12, 1, True), (1000, 4, 12, 1, True), (256, 12, 12, 1, True),  # 44, 11.5; 80, 71
    (40, 12, 1, 1, True), (300, 3, 5, 7, True), (1000, 8, 9, 4, True),
    (1000, 12, 1, 1, False), (1000, 12, 1, 7, False),                     # 12.1, 49; 32.7, 325
    (300, 10, 3, 4, False), (1000, 10, 7, 4, False),                      # 17, 34; 99, 138
    (3000, 4, 1, 7, False), (300, 16, 1, 1, False),
])
def test_kernel_of_uniform_orders(host, B, M, N, R, few):
    h = host.tables(uniform(B, M, N))
    size = host.lib.mudiff_matvec_workspace_size(h, R)
    host.launches.clear()
    host.check(host.lib.mudiff_matvec(h, R, 256, 512, 1, 1024, size, None))
    names = [n for n, *_ in host.launches]
    assert ("k_apply_few" in names[0]) == few and len(names) == (1 if few else 2), names
    host.check(host.lib.mudiff_destroy(h))


@pytest.mark.parametrize("instances,R,restart,small", [
    # (us of a step as three kernels and in one workgroup)
    (uniform(1, 4, 15), 1, 30, True), (uniform(1, 12, 12), 1, 30, True),          # 22.8, 19.4
    (uniform(10, 8, 15), 4, 40, True), (batch([12] * 64, 5, 18), 7, 30, True),
    (uniform(300, 12, 12), 7, 20, True), (uniform(256, 4, 12), 7, 30, True),
    (uniform(1, 8, 25), 1, 30, True), (uniform(270, 16, 12), 7, 30, True),
    (uniform(1, 16, 12), 1, 10, False), (uniform(1, 16, 15), 4, 10, False),       # 16.5, 21.4
    (batch([16] * 10, 5, 18), 1, 10, False), (uniform(1, 11, 16), 1, 10, False),  # 14.2, 18.1; 24.8, 29.6
    (uniform(300, 16, 1), 7, 20, False), (uniform(300, 13, 3), 7, 20, False),     # 75, 149; 93, 125
    (uniform(64, 16, 1), 7, 20, False),                                           # 29, 41
    (uniform(16, 16, 12), 4, 24, False), (uniform(1, 12, 15), 1, 30, True),       # 31.5, 34.7; 26.5, 23.5
])
def test_cycles_of_small_columns(host, instances, R, restart, small):
    """The kernels of a solve's first cycle; its state reads as running until one of them is launched,
    then as ended."""
    h = host.tables(instances)
    B = len(instances)
    size = host.lib.mudiff_gmres_workspace_size(h, R, restart, 0)
    ws, out = host.array(size), host.array(B * R * 16 + 4096)
    ws.data[:] = 1
    ended = lambda read, blocks: ws.data.fill(0)  # noqa: E731
    host.hooks = {"k_small_cycle": ended, "k_dg_dots": ended}
    host.launches.clear()
    host.check(host.lib.mudiff_gmres(h, R, 256, None, 512, restart, 1e-8, 1000, 0, ws.base, size, out.base, out.base,
                                     out.base, None, None))
    host.hooks = {}
    names = {n for n, *_ in host.launches}
    assert any("k_small_cycle" in n for n in names) == small, names
    assert any("k_dg_update" in n for n in names) != small, names
    host.check(host.lib.mudiff_destroy(h))


@pytest.mark.parametrize("B,M,N,rows", [
    # (four rows per workgroup over one, in time)
    (1, 400, 12, 4), (1, 700, 9, 4), (100, 64, 10, 4),    # 0.91 to 0.96
    (1, 400, 8, 1), (1, 700, 7, 1), (1, 300, 1, 1),       # 1.00 to 1.3
    (300, 17, 12, 1), (300, 22, 9, 1), (100, 13, 11, 1),  # 1.15, 1.09, 1.2: groups of 1 to 3 rows
    (300, 20, 12, 4), (1, 100, 12, 1),                    # 200 waves
])
def test_rows_per_workgroup(host, B, M, N, rows):
    h = host.tables(uniform(B, M, N))
    size = host.lib.mudiff_matvec_workspace_size(h, 7)
    host.launches.clear()
    host.check(host.lib.mudiff_matvec(h, 7, 256, 512, 1, 1024, size, None))
    (name, _, threads, _, _), *_ = host.launches
    assert "k_apply_lane" in name and threads == 64 * rows, (name, threads)
    host.check(host.lib.mudiff_destroy(h))
