"""CC by union-find where most of the work lies outside the giant component:
rows around the heavy threshold and the chunk size there, a hub whose
neighbours are trees of their own, two skewed components of one size -- against the
oracle, and no slower than a few edge sweeps take.
"""
import time

import numpy as np
import pytest

import oracle
from paper_1903_01665_amd import gen

pytestmark = pytest.mark.gpu


def join(name, *parts):
    """The parts (n, src, dst) side by side, each with the ids after the last one's."""
    base, src, dst = 0, [], []
    for n, s, d in parts:
        src.append(np.asarray(s, np.int64) + base)
        dst.append(np.asarray(d, np.int64) + base)
        base += n
    s, d = (np.concatenate(x).astype(np.int32) for x in (src, dst))
    return gen.from_edges(base, s, d, np.ones(len(s), np.int32), name=name)


def uniform(n, m, seed):
    rng = np.random.default_rng(seed)
    return n, rng.integers(0, n, m), rng.integers(0, n, m)


def star(leaves, hub_first=False):
    """The hub has the largest id, so that most leaves stay trees of their own."""
    if hub_first:
        return leaves + 1, np.zeros(leaves, int), 1 + np.arange(leaves)
    return leaves + 1, np.full(leaves, leaves), np.random.default_rng(leaves).permutation(leaves)


def rmat(scale, stream):
    h = gen.rmat(scale, 8 << scale, stream=stream)
    return h.n, np.repeat(np.arange(h.n), np.diff(h.row_ptr)), h.col


def graphs():
    giant = uniform(30000, 120000, 1)
    sizes = [1, 15, 16, 17, 31, 32, 33, 127, 128, 129, 255, 256, 257, 4097]
    return [join("rows", giant, *[star(k) for k in sizes], *[star(k, True) for k in sizes]),
            join("hub", giant, star(9000)), join("two-rmat", rmat(13, 501), rmat(13, 502)),
            join("hubs-linked", giant, (4002, np.r_[np.full(2000, 4000), np.full(2000, 4001), 4000],
                                        np.r_[np.arange(4000), 4001]))]


@pytest.mark.parametrize("hg", graphs(), ids=lambda h: h.name)
def test_cc_outside_the_giant(hg):
    from paper_1903_01665_amd import gg
    want = oracle.cc(hg.n, hg.row_ptr, hg.col)
    for renumber in (False, True):
        g = gg.Graph.from_host(hg, symmetrize=True, renumber=renumber)
        try:
            for cap in (0, 1, 3):
                print(hg.name, renumber, cap, flush=True)
                o = gg.make_opts(gg.VERTEX, gg.UNIONFIND, max_blocks=cap)
                for _ in range(3):
                    np.testing.assert_array_equal(g.cc(opts=o).cpu().numpy(), want)
        finally:
            g.free()


def best_ms(f):
    import torch
    times = []
    for _ in range(6):
        t = time.perf_counter()
        f()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
    return 1e3 * min(times)


@pytest.mark.parametrize("shape", ["skewed", "chain", "shuffled-chain"])
def test_cc_has_no_serial_path(shape):
    """Edge sweeps take a few passes on the skewed graph; the passes over a chain
    are gathers of its parents, tens of microseconds each."""
    import torch

    from paper_1903_01665_amd import gg
    if shape == "skewed":
        hg = join(shape, rmat(17, 503), rmat(17, 504), star(1 << 18))
    else:
        p = np.arange(1 << 20)
        if shape != "chain":
            p = np.random.default_rng(9).permutation(p)
        hg = join(shape, (len(p), p[:-1], p[1:]))
    g = gg.Graph.from_host(hg, symmetrize=True)
    out = torch.empty(hg.n, dtype=torch.int32, device="cuda")
    try:
        uf = best_ms(lambda: g.cc(opts=gg.make_opts(gg.VERTEX, gg.UNIONFIND), out=out))
        np.testing.assert_array_equal(out.cpu().numpy(), oracle.cc(hg.n, hg.row_ptr, hg.col))
        limit = 1.0  # ms: 2^20 vertices, twenty passes of 50 us
        if shape == "skewed":
            limit = 4 * best_ms(lambda: g.cc(opts=gg.make_opts(gg.EDGE, gg.SYNC), out=out))
        print(shape, uf, limit, flush=True)
        assert uf < limit
    finally:
        g.free()
