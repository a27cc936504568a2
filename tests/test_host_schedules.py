"""Schedules of the operator apply on the host alone (tests/native/build_host.py: kernels are
recorded, not run): what the launches are given lies inside the workspace whose size the library
asks for, for every tile that the setters can lead to."""
import ctypes
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "native"))
import build_host  # noqa: E402


@pytest.fixture(scope="module")
def host():
    return build_host.Host()


def grid(M, spacing, orders, k=5.0):
    """M unit disks on a square grid, with orders taken in turn."""
    w = int(np.ceil(np.sqrt(M)))
    c = np.array([(i % w, i // w) for i in range(M)], float) * spacing
    return c, np.ones(M), np.resize(orders, M), k


ORDERS = [16, 23, 19, 21]


def mixed(M, m):
    """A sparse instance of M disks (in the circulant form) and a dense one of m (outside it:
    all its pairs are close)."""
    return [grid(M, 10.0, ORDERS), grid(m, 2.1, ORDERS)]


class Applies:
    """Applies of one handle, each in a workspace of the size that the library names; notes the
    largest end of the work queue's partial sums, relative to that workspace."""

    def __init__(self, host, h, R):
        self.host, self.h, self.R = host, h, R
        n = (ctypes.c_int64 * 512)()  # unknowns of every instance
        host.check(host.lib.mudiff_sizes(h, n))
        self.x = host.array(16 * R * sum(n))
        self.y = host.array(16 * R * sum(n))
        self.bytes = host.lib.mudiff_matvec_workspace_size(h, R)
        self.ws = host.array(self.bytes)
        self.end, self.queues = 0, 0
        host.hooks["k_apply_mfmaI"] = self.queue

    def queue(self, read, blocks):
        # (view, R, x, active, items, n_items, head, part, blk, ...)
        n = read(5, ctypes.c_int32)
        items = np.ctypeslib.as_array(ctypes.cast(read(4, ctypes.c_void_p), ctypes.POINTER(ctypes.c_int32)), (n, 7))
        part, blk = read(7, ctypes.c_void_p), read(8, ctypes.c_int64)
        self.end = max(self.end, part + (int(items[:, 5].max()) + 1) * blk * 16 - self.ws.base)
        self.queues += 1

    def run(self):
        self.host.check(self.host.lib.mudiff_matvec(self.h, self.R, self.x.base, self.y.base, 1,
                                                    self.ws.base, self.bytes, None))
        assert self.end <= self.bytes, (self.end, self.bytes)

    def tile(self):
        v = [ctypes.c_int(0) for _ in range(6)]
        self.host.check(self.host.lib.mudiff_circulant_tile(self.h, self.R, *[ctypes.byref(x) for x in v]))
        return [x.value for x in v]

    def config(self):
        v = [ctypes.c_int(0) for _ in range(5)]
        self.host.check(self.host.lib.mudiff_apply_config(self.h, self.R, *[ctypes.byref(x) for x in v], None))
        return [x.value for x in v]


@pytest.mark.parametrize("M,m,R", [(200, 10, 64), (400, 20, 32), (60, 17, 9), (90, 3, 130)])
def test_partial_sums_inside_the_workspace_when_the_form_changes(host, M, m, R):
    """A timed choice of the circulant form, its tile fixed, the form switched off and on again:
    the work queue's segments suit the form that runs."""
    h = host.tables(mixed(M, m), circulant=True)
    lib = host.lib
    for first in (0, 1):  # the first candidate (circulant form) or the last one (direct) is the fastest
        a = Applies(host, h, R)
        t = iter(range(1000, 0, -1))
        host.clock(lambda: float(next(t)) if first else 1.0)
        host.check(lib.mudiff_set_circulant(h, R, -1))
        a.run()
        if a.config()[0] == 3:
            host.check(lib.mudiff_set_circulant_tile(h, R, *a.tile()))
            a.run()
        host.check(lib.mudiff_set_circulant(h, R, 0))
        a.run()
        host.check(lib.mudiff_set_circulant(h, R, 1))
        a.run()
        for ct in (1, 2, 4):  # direct tiles that a caller may fix, in both forms
            for waves in (4, 8):
                for qs in (0, 32):
                    if ct > max(1, -(-R // 8)):
                        continue
                    if lib.mudiff_set_apply_config(h, R, ct, waves // ct, qs, 64 * waves):
                        continue
                    for mode in (1, 0):
                        host.check(lib.mudiff_set_circulant(h, R, mode))
                        a.run()
        assert a.queues > 0
    host.check(lib.mudiff_destroy(h))


@pytest.mark.parametrize("R", [8, 64])
def test_second_stream_only_outside_captures_and_profiles(host, R):
    """A batch with a short queue beside the circulant form: the queue runs on the handle's second
    stream, but not while the caller captures the apply or an apply is profiled (its phases are
    timed between events of the caller's stream)."""
    h = host.tables(mixed(200, 10), circulant=True)
    host.clock(lambda: 1.0)
    a = Applies(host, h, R)
    a.run()

    def streams():
        host.launches.clear()
        n = a.queues
        a.run()
        assert a.queues == n + 1  # a queue there is
        return {s for *_, s in host.launches}

    assert len(streams()) == 2
    host.lib.host_capturing(1)
    assert streams() == {None}
    host.lib.host_capturing(0)
    host.check(host.lib.mudiff_profile_begin(h, 1))
    assert streams() == {None}
    assert len(streams()) == 2  # past the profiled applies
    n, ms = ctypes.c_int(0), (ctypes.c_double * 5)()
    host.check(host.lib.mudiff_profile_end(h, ctypes.byref(n), ms))
    assert n.value == 1
    host.check(host.lib.mudiff_destroy(h))


def pick(host, win):
    """Clock under which timed candidate number `win` is the fastest."""
    n = iter(range(10 ** 6))
    host.clock(lambda: 1.0 if next(n) == win else 2.0)


def test_timed_product_tiles_can_be_fixed(host):
    """Every product tile that first use may choose is one that set_circulant_tile takes, and that
    Problem.circulant_tiles lists."""
    from paper_1409_8186_amd.api import Problem
    h = host.tables([grid(30, 10.0, ORDERS)], circulant=True)
    for R in range(8, 70):
        seen = set()
        for win in range(6):  # timed pairs, and the warm-ups between them
            host.check(host.lib.mudiff_set_circulant(h, R, 1))
            pick(host, win)
            a = Applies(host, h, R)
            a.run()
            seen.add(tuple(a.tile()))
            # timed again at the next round: back to no choice
            host.check(host.lib.mudiff_set_circulant(h, R, 1))
        for t in seen:
            assert t in Problem.circulant_tiles(R), (R, t)
        for t in Problem.circulant_tiles(R):
            host.check(host.lib.mudiff_set_circulant_tile(h, R, *t))
        host.check(host.lib.mudiff_destroy(h))
        h = host.tables([grid(30, 10.0, ORDERS)], circulant=True)
    host.check(host.lib.mudiff_destroy(h))


@pytest.mark.parametrize("instances", [[grid(30, 10.0, ORDERS)], [grid(30, 2.1, [8, 3])], mixed(50, 10)],
                         ids=["sparse", "dense", "mixed"])
def test_timed_configuration_can_be_fixed(host, instances):
    """What apply_config reports of a timed apply is taken by set_apply_config, here and on another
    handle of the same batch, and reported again; other lengths are refused."""
    for R in (8, 11, 16, 24, 33, 64):
        for win in range(10):
            pick(host, win)
            h = host.tables(instances, circulant=True)
            Applies(host, h, R).run()
            a = Applies(host, h, R)
            found = a.config()
            host.check(host.lib.mudiff_destroy(h))
            h = host.tables(instances, circulant=True)
            a = Applies(host, h, R)
            for _ in range(2):
                host.check(host.lib.mudiff_set_circulant(h, R, int(found[0] == 3)))
                host.check(host.lib.mudiff_set_apply_config(h, R, *found[1:]))
                assert a.config() == found
                a.run()
            for qs in (1, 5, 31, 128):
                assert host.lib.mudiff_set_apply_config(h, R, *found[1:3], qs, found[4]) == 1
            assert a.config() == found
            host.check(host.lib.mudiff_destroy(h))


@pytest.mark.parametrize("instances,R,timed", [
    ([grid(12, 2.1, ORDERS)] * 8, 20, {0, 4}), ([grid(200, 2.1, [31])], 20, {0, 8, 16, 32}),
    ([grid(6, 2.1, ORDERS)] * 300, 12, {0, 4}), ([grid(20, 2.1, ORDERS)] * 64, 20, {0, 16}),
], ids=["8x12", "200", "300x6", "64x20"])
def test_segments_that_are_timed(host, instances, R, timed):
    """Each tile of the direct form that first use times is timed with the rule's segment length, with
    whole instances and with segments of 32."""
    seen = set()
    for win in range(18):
        pick(host, win)
        h = host.tables(instances)
        a = Applies(host, h, R)
        a.run()
        seen.add(tuple(a.config()[1:4]))
        host.check(host.lib.mudiff_destroy(h))
    assert {qs for *_, qs in seen} == timed
    tiles = {(ct, rp) for ct, rp, _ in seen}
    assert all({qs for c, r, qs in seen if (c, r) == t} >= {0} | ({32} & timed) for t in tiles), seen
