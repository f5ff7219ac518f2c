"""Static components on graphs where hooking makes long chains, many trees or none: paths whose
ids rise, fall or are shuffled, combs and grids, many small components beside none that is large,
and components of nearly equal size; with the undirected view and without it."""
import numpy as np
import pytest

from paper_2305_17813_amd import inputs as I
from paper_2305_17813_amd import native
from parity import Pair, say

pytestmark = pytest.mark.gpu


def path(n, order):
    ids = {"rising": np.arange(n), "falling": np.arange(n)[::-1],
           "shuffled": np.random.default_rng(3).permutation(n)}[order]
    ids = np.ascontiguousarray(ids)
    return ids[:-1], ids[1:], n


def cliques(count, size):
    a, b = np.triu_indices(size, 1)
    base = np.arange(count)[:, None] * size
    return (base + a).ravel(), (base + b).ravel(), count * size + 3


def comb(teeth, length):
    """A path of `teeth` vertices, each with a path of `length` hanging off it."""
    s, d, _ = path(teeth, "falling")
    first = teeth + np.arange(teeth) * length
    s, d = [s, np.arange(teeth)], [d, first]
    for k in range(length - 1):
        s.append(first + k)
        d.append(first + k + 1)
    return np.concatenate(s), np.concatenate(d), teeth * (length + 1)


def grid(side):
    g = I.grid_graph(side, 5)
    return g.src.numpy(), g.dst.numpy(), g.n


def two_stars(leaves):
    n = 2 * leaves + 2
    s = np.concatenate([np.full(leaves, n - 1), np.full(leaves, n - 2)])
    return s, np.arange(2 * leaves), n


CASES = {
    "rising path": path(5000, "rising"), "falling path": path(5000, "falling"),
    "shuffled path": path(5000, "shuffled"), "pairs": cliques(3000, 2), "cliques of 5": cliques(700, 5),
    "comb": comb(300, 20), "grid": grid(70), "two stars": two_stars(2500),
}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("views", [native.VIEW_FWD, native.VIEW_FWD | native.VIEW_REV, 7])
def test_components(name, views):
    say(f"case: components, {name}, views {views}")
    s, d, n = CASES[name]
    p = Pair(n, s, d, np.ones(len(s), np.int64), views=views)
    p.check_wcc()
    cut = np.ascontiguousarray(s[::7]), np.ascontiguousarray(d[::7])
    p.delete(*cut)  # tombstones in the first words; a recompute
    p.check_wcc()
    p.insert(*cut, np.ones(len(cut[0]), np.int64))  # incremental on the recomputed forest
    p.check_wcc()
    p.check_wcc(native.RECOMPUTE)


# without the undirected view: vertices of several buckets on either side of the sizes from and to
# which trees are hooked before the walk (2^15 and 2^19 vertices), and the smallest sizes
@pytest.mark.parametrize("n,extra", [(900, 40), (32_767, 30), (32_768, 30), (524_288, 12), (524_289, 12)])
def test_all_arc_walk(n, extra):
    say(f"case: components by the all-arc walk, {n} vertices")
    rng = np.random.default_rng(n)
    hubs = rng.choice(n, 50, replace=False)
    s = np.concatenate([rng.integers(0, n, n // 3), np.repeat(hubs, extra)])
    d = rng.integers(0, n, len(s))
    key = np.unique(s * n + d)
    s, d = key // n, key % n
    s, d = s[s != d], d[s != d]
    p = Pair(n, s, d, np.ones(len(s), np.int64), views=native.VIEW_FWD)
    p.check_wcc()
    p.check_wcc(native.RECOMPUTE)
    p.delete(s[::5], d[::5])
    p.check_wcc()
    p.insert(s[::5], d[::5], np.ones(len(s[::5]), np.int64))
    p.check_wcc()


# graphs of few neighbours a vertex take the all-arc walk; with long chains allowed, or filled by
# inserts, they are sampled like any other
@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("filled", [False, True])
def test_sampled_components_of_the_same_graphs(name, filled):
    say(f"case: components, {name}, sampled, filled by inserts {filled}")
    s, d, n = CASES[name]
    w = np.ones(len(s), np.int64)
    k = 0 if filled else len(s)
    p = Pair(n, s[:k], d[:k], w[:k], load_factor=0.7 if filled else 2.0)
    if filled:
        p.insert(s, d, w, exact_status=False)
    p.check_wcc()
    cut = np.ascontiguousarray(s[::7]), np.ascontiguousarray(d[::7])
    p.delete(*cut, exact_status=False)
    p.check_wcc()
    p.insert(*cut, np.ones(len(cut[0]), np.int64), exact_status=False)
    p.check_wcc()
    p.check_wcc(native.RECOMPUTE)


# graphs most of whose vertices have no arc (those are not sampled), down to no arc at all
@pytest.mark.parametrize("n,among,arcs", [(1, 1, 0), (300, 2, 0), (5000, 2, 1), (5000, 40, 25), (40_000, 900, 1500),
                                          (200_000, 70_000, 140_000)])
def test_sampled_components_among_vertices_without_arcs(n, among, arcs):
    say(f"case: components, {arcs} arcs among {among} of {n} vertices")
    rng = np.random.default_rng(n + arcs)
    ids = np.sort(rng.choice(n, among, replace=False))
    s, d = rng.integers(0, among, arcs), rng.integers(0, among, arcs)
    d = np.where(s == d, (d + 1) % among, d)
    key = np.unique(ids[s] * n + ids[d])
    s, d = key // n, key % n
    p = Pair(n, s, d, np.ones(len(s), np.int64), load_factor=2.0)
    p.check_wcc()
    if arcs:
        p.delete(s[::2], d[::2])
        p.check_wcc()
        p.delete(s[1::2], d[1::2])  # no arc left
        p.check_wcc()
        for half in (slice(0, None, 2), slice(1, None, 2)):  # the slab pool has room for either
            p.insert(s[half], d[half], np.ones(len(s[half]), np.int64))
            p.check_wcc()
        p.check_wcc(native.RECOMPUTE)


# the walk over graphs without vertices of several buckets, whose blocks grow with the root of the
# vertices: the smallest, and sizes whose blocks take several rounds with a ragged last one
@pytest.mark.parametrize("views", [native.VIEW_FWD, native.VIEW_FWD | native.VIEW_REV])
@pytest.mark.parametrize("n", [1, 2, 257, 16_385, 70_001, 1_100_003])
def test_all_arc_walk_of_single_buckets(n, views):
    say(f"case: components by the all-arc walk, {n} vertices of one bucket, views {views}")
    rng = np.random.default_rng(n)
    ring = np.arange(n)
    s = np.concatenate([ring[: n // 2], rng.integers(0, n, n // 4)])
    d = np.concatenate([ring[: n // 2] + 1, rng.integers(0, n, n // 4)]) % n
    key = np.unique(s * n + d)
    s, d = key // n, key % n
    s, d = s[s != d], d[s != d]
    p = Pair(n, s, d, np.ones(len(s), np.int64), views=views, load_factor=0.0)
    p.check_wcc()
    p.check_wcc(native.RECOMPUTE)
    if len(s):
        p.delete(s[::9], d[::9])
        p.check_wcc()
        p.insert(s[::9], d[::9], np.ones(len(s[::9]), np.int64))
        p.check_wcc()
