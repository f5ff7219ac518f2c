"""The static triangle count at the edges of its vertex classes, against closed forms."""
from math import comb

import numpy as np
import pytest
import torch

from paper_2305_17813_amd import inputs as I
from paper_2305_17813_amd import native
from parity import Pair, say

pytestmark = pytest.mark.gpu


# K_n has vertices of every out-degree below n in the degree order: around the wave class's 64
# keys, the 256-thread class's 640 and one pass of the largest class (5,120 keys)
@pytest.mark.parametrize("n", [3, 64, 65, 66, 67, 640, 641, 642, 5200])
def test_complete_graph(n):
    say(f"case: static triangles of K_{n}")
    u, v = torch.triu_indices(n, n, 1, device="cuda")
    views = native.VIEW_FWD | native.VIEW_UND
    g = native.Graph(n + 2, u, v, views=views)  # and two isolated vertices
    assert int(g.triangles(mode=native.RECOMPUTE).item()) == comb(n, 3)
    if n <= 642:  # a vertex joined to all, then one edge gone: exact after updates and recounts
        s = torch.full((n,), n, device="cuda")
        g.insert_edges(s, torch.arange(n, device="cuda"))
        assert int(g.triangles().item()) == comb(n + 1, 3)
        assert int(g.triangles(mode=native.RECOMPUTE).item()) == comb(n + 1, 3)
        g.delete_edges(s[:1], torch.zeros(1, dtype=torch.int64, device="cuda"))
        assert int(g.triangles(mode=native.RECOMPUTE).item()) == comb(n + 1, 3) - (n - 1)


@pytest.mark.parametrize("load_factor", [0.7, 0.0])
def test_power_law_graph_with_long_chains(load_factor):
    """Against the oracle, with hashing on and off (chains of many slabs) and tombstones; a
    repeated call without a pending batch, with other calls between, repeats its answer."""
    say(f"case: static triangles, load factor {load_factor}")
    g = I.rmat_s(11)
    p = Pair(g.n, g.src, g.dst, g.w, load_factor=load_factor)
    p.check_tc()
    s, d = I.Workload(g, 3).delete_batch(2000)
    p.delete(s, d)
    p.check_tc()
    p.g.stats()
    p.check_tc()
    p.check_tc(native.RECOMPUTE)


# vertices whose buckets outlive their arcs: a lane's, a group's, a block's (17 buckets) and several
# rounds of a block's chains; their lists must stay empty and leave their neighbours' lists alone
@pytest.mark.parametrize("degree", [1, 60, 160, 190, 1000, 4000])
@pytest.mark.parametrize("everything", [False, True])
def test_vertices_that_lost_all_their_arcs(degree, everything):
    """Every arc of three such vertices is deleted, once one by one and once with all others of
    the graph; the vertices with neighbouring ids keep their triangles."""
    say(f"case: static triangles, {degree} deleted arcs of a vertex, everything {everything}")
    n = degree + 40
    hubs = [4, 5, 20]
    u, v = np.triu_indices(24, 1)  # K_24 on the first vertices, the hubs among them
    s, d = [u], [v]
    for h in hubs:
        leaf = 24 + np.arange(degree)
        s.append(np.full(degree, h))
        d.append(leaf)
    s, d = np.concatenate(s), np.concatenate(d)
    p = Pair(n, s, d, np.ones(len(s), np.int64), views=native.VIEW_FWD | native.VIEW_UND)
    p.check_tc(native.RECOMPUTE)
    gone = np.isin(s, hubs) | np.isin(d, hubs) | everything
    p.delete(np.ascontiguousarray(s[gone]), np.ascontiguousarray(d[gone]))
    p.check_tc(native.RECOMPUTE)  # among tombstones
    p.g.compact()
    p.check_tc(native.RECOMPUTE)  # among empty words
    p.insert(np.ascontiguousarray(s[gone]), np.ascontiguousarray(d[gone]), np.ones(int(gone.sum()), np.int64))
    p.check_tc()
    p.check_tc(native.RECOMPUTE)


@pytest.mark.parametrize("n", [3, 66, 642])
def test_complete_graph_filled_by_inserts(n):
    """Classes that the arcs of creation alone could not fill."""
    say(f"case: static triangles of K_{n}, filled by inserts")
    u, v = torch.triu_indices(n, n, 1, device="cuda")
    none = torch.zeros(0, dtype=torch.int32, device="cuda")
    g = native.Graph(n + 2, none, none, views=native.VIEW_FWD | native.VIEW_UND, pool_slabs=1 << 20)
    assert int(g.triangles(mode=native.RECOMPUTE).item()) == 0
    g.insert_edges(u, v)
    assert int(g.triangles(mode=native.RECOMPUTE).item()) == comb(n, 3)
    g.delete_edges(u, v)
    assert int(g.triangles(mode=native.RECOMPUTE).item()) == 0


def test_replayed_recount_follows_the_graph():
    """A captured recount is replayed on a graph that grows out of the classes it was captured with,
    with eager work between the replays."""
    say("case: static triangles, captured")
    n = 700
    u, v = torch.triu_indices(n, n, 1, device="cuda")
    order = torch.randperm(len(u), generator=torch.Generator().manual_seed(3)).cuda()
    u, v = u[order], v[order]
    g = native.Graph(n, u[:100], v[:100], views=native.VIEW_FWD | native.VIEW_UND, pool_slabs=1 << 20)
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        count.copy_(g.triangles(mode=native.RECOMPUTE, stream=stream))
    done = 100
    for k in (100, 1200, 40_000, len(u), len(u)):
        if k > done:
            g.insert_edges(u[done:k], v[done:k])
            done = k
        graph.replay()
        torch.cuda.synchronize()
        got = int(count.item())
        assert got == int(g.triangles(mode=native.RECOMPUTE).item())
        assert int(g.stats()["n_und_edges"]) == done
    assert got == comb(n, 3)


# degrees that buckets and arcs inserted since keep at 64 or below are counted without lists
@pytest.mark.parametrize("inserted", [0, 30, 200])
def test_lattice(inserted):
    say(f"case: static triangles of a lattice, {inserted} arcs inserted")
    side = 45
    v = np.arange(side * side).reshape(side, side)
    s = np.concatenate([v[:, :-1].ravel(), v[:-1].ravel(), v[:-1, :-1].ravel()])
    d = np.concatenate([v[:, 1:].ravel(), v[1:].ravel(), v[1:, 1:].ravel()])
    p = Pair(side * side, s, d, np.ones(len(s), np.int64))
    p.check_tc()
    p.delete(s[::9], d[::9])
    p.check_tc(native.RECOMPUTE)
    if inserted:  # a hub beside the lattice
        p.insert(np.full(inserted, 3), 100 + np.arange(inserted), np.ones(inserted, np.int64), exact_status=False)
        p.check_tc(native.RECOMPUTE)
    p.g.compact()
    p.check_tc(native.RECOMPUTE)
    p.delete(s, d)
    p.check_tc(native.RECOMPUTE)


# a stream of batches that come and go leaves a graph of few neighbours what it was: counts and
# components before, between and after them, by any way of laying the chains
@pytest.mark.parametrize("load_factor", [0.7, 2.0, 0.0])
@pytest.mark.parametrize("batch", [40, 1500])
def test_streams_over_a_lattice(load_factor, batch):
    say(f"case: recounts along a stream over a lattice, batches of {batch}, load factor {load_factor}")
    side = 40
    v = np.arange(side * side).reshape(side, side)
    s = np.concatenate([v[:, :-1].ravel(), v[:-1].ravel(), v[:-1, :-1].ravel()])
    d = np.concatenate([v[:, 1:].ravel(), v[1:].ravel(), v[1:, 1:].ravel()])
    p = Pair(side * side, s, d, np.ones(len(s), np.int64), load_factor=load_factor)
    rng = np.random.default_rng(batch)
    for k in range(5):
        a = rng.integers(0, side * side, batch)
        b = np.full(batch, 7 + k) if batch < 100 else rng.integers(0, side * side, batch)  # one vertex, or all
        key = np.unique(a * side * side + b)
        a, b = key // (side * side), key % (side * side)
        new = (a != b) & ~np.isin(a * side * side + b, s * side * side + d)
        a, b = a[new], b[new]
        p.insert(a, b, np.ones(len(a), np.int64))
        p.check_tc(native.RECOMPUTE)
        p.check_wcc(native.RECOMPUTE)
        p.delete(a, b)
        p.check_tc(native.RECOMPUTE)
        p.check_wcc(native.RECOMPUTE)
    assert p.g.check() == 0
