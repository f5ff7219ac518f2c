"""Compaction by the logged deletes and by a sweep over every chain give the same graph."""
import numpy as np
import pytest
import torch

from paper_2305_17813_amd import inputs as I
from paper_2305_17813_amd import native
from parity import Pair, say, u32

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("views", [1, 3, 5, 7])
@pytest.mark.parametrize("load_factor", [0.7, 0.0])
def test_logged_deletes_and_full_sweep_agree(views, load_factor):
    """Two copies of a graph take the same batches.  One copy's change log holds every batch
    (the logged deletes' chains are visited), the other's only the last one (every chain is
    swept).  Both free the same number of slabs, leave no tombstone behind and hold the
    oracle's arcs; batches with repeated arcs, absent arcs and both directions of an edge are
    among them, and thresholds above one come before a threshold of one."""
    say(f"case: compaction paths, views {views}, load factor {load_factor}")
    g = I.rmat_s(11)
    s0, d0, w0 = g.src, g.dst, g.w
    # both copies build in chunks that fit their logs; chunking does not change what a chain holds
    a = Pair(g.n, s0, d0, w0, views=views, load_factor=load_factor, log_capacity=1 << 20)
    b = Pair(g.n, s0, d0, w0, views=views, load_factor=load_factor, log_capacity=4001)
    rng = np.random.default_rng(5)
    arcs = np.stack([s0.numpy(), d0.numpy()], 1)
    for thresholds in ([3, 1], [1, 1], [2, 1]):
        picks = arcs[rng.permutation(len(arcs))[:3000]]
        batch1 = np.concatenate([picks[:2000], picks[:500, ::-1], picks[:200]])  # reversed and repeated arcs
        batch2 = picks[1500:]
        for p in (a, b):
            for q in (batch1, batch2):
                p.delete(torch.as_tensor(q[:, 0].copy()), torch.as_tensor(q[:, 1].copy()), exact_status=False)
        for t in thresholds:
            fa, fb = a.g.compact(t), b.g.compact(t)
            assert fa == fb, (fa, fb)
            assert a.g.stats()["pool_used"] == b.g.stats()["pool_used"]
        assert a.g.compact() == 0
        a.check_structure()
        b.check_structure()
        w = torch.as_tensor(I.arc_weight(torch.as_tensor(picks[:, 0].copy()), torch.as_tensor(picks[:, 1].copy()),
                                         g.wmax, g.wseed))
        for p in (a, b):
            p.insert(torch.as_tensor(picks[:, 0].copy()), torch.as_tensor(picks[:, 1].copy()), w)
    a.check_all(algos=("bfs", "sssp", "wcc"))


def test_replayed_deletes_are_reclaimed():
    """A captured delete that is replayed with other arcs leaves tombstones the log does not
    name: compaction sweeps every chain then, and reclaims all of them."""
    say("case: compaction after replayed deletes")
    n = 2000
    dst = np.arange(1, 1801)
    p = Pair(n, np.zeros(1800, np.int64), dst, np.full(1800, 3), load_factor=0.0, views=native.VIEW_FWD)
    s = torch.zeros(600, dtype=torch.int32, device="cuda")
    d = torch.as_tensor(dst[:600], dtype=torch.int32, device="cuda")
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        p.g.delete_edges(s, d, status=False, stream=stream)
    for k in range(2):  # deletes 1..600, then 601..1200
        d.copy_(torch.as_tensor(dst[600 * k:600 * (k + 1)], dtype=torch.int32))
        graph.replay()
        torch.cuda.synchronize()
        p.o.delete(np.zeros(600, np.uint32), dst[600 * k:600 * (k + 1)].astype(np.uint32))
    # one chain of 120 slabs keeps 600 arcs: 40 slabs, the head among them
    assert p.g.compact() == 80
    p.check_structure()
    assert p.g.compact() == 0


# ops per batch (two batches, among them repeated, reversed and absent arcs) on graphs of 2^scale
# vertices; from 16,384 ops on, a block takes several chains a group
@pytest.mark.parametrize("views,scale,ops,load_factor", [
    (1, 14, 1, 0.7), (1, 14, 900, 0.7), (3, 14, 1500, 0.7), (5, 14, 1900, 0.7), (7, 14, 2500, 0.7),
    (1, 14, 1, 0.0), (1, 14, 900, 0.0), (3, 14, 1500, 0.0), (5, 14, 1900, 0.0), (7, 14, 2500, 0.0),
    (7, 18, 16_000, 0.7), (7, 18, 40_000, 0.7)])
def test_chains_of_logged_deletes(views, scale, ops, load_factor):
    """A copy whose log holds every delete, few enough of them, against one whose log lost the first
    batch (a sweep) and against the oracle."""
    say(f"case: logged compaction, views {views}, {ops} ops, load factor {load_factor}")
    g = I.rmat_graph(scale, 8, 31)
    s0, d0, w0 = (np.asarray(x.cpu()).view(np.uint32).astype(np.int64) for x in g.u32())
    a = Pair(g.n, s0, d0, w0, views=views, load_factor=load_factor)
    b = Pair(g.n, s0, d0, w0, views=views, load_factor=load_factor, log_capacity=max(2, ops))
    rng = np.random.default_rng(ops)
    arcs = np.stack([s0, d0], 1)
    for thresholds in ([1], [3, 2, 1]):
        picks = arcs[rng.permutation(len(arcs))[:ops]]
        batch1 = np.concatenate([picks[: ops // 2], picks[: ops // 5, ::-1], picks[: ops // 9]])
        batch2 = picks[ops // 3:]
        logged = len(batch1) + len(batch2)
        assert 8 * logged <= sum(a.g.stats()["head_slabs"]), "the first copy must go by its log"
        for p in (a, b):
            for q in (batch1, batch2):
                p.delete(q[:, 0].copy(), q[:, 1].copy(), exact_status=False)
            if logged <= max(2, ops):  # one more batch takes the first one's place in the second copy's log
                for _ in range(3):
                    p.delete(batch2[:1, 0].copy(), batch2[:1, 1].copy(), exact_status=False)
        for t in thresholds:
            fa, fb = a.g.compact(t), b.g.compact(t)
            assert fa == fb, (fa, fb)
            assert a.g.stats()["pool_used"] == b.g.stats()["pool_used"]
        assert a.g.compact() == 0 and b.g.compact() == 0
        a.check_structure()
        b.check_structure()
        for p in (a, b):
            p.insert(s0[:0], d0[:0], w0[:0])
            p.insert(picks[:, 0].copy(), picks[:, 1].copy(),
                     u32(I.arc_weight(torch.as_tensor(picks[:, 0].copy()), torch.as_tensor(picks[:, 1].copy()), g.wmax,
                                      g.wseed)).astype(np.int64))
        a.check_structure()
    a.check_all(algos=("wcc", "tc"))


@pytest.mark.parametrize("more", [0, 1])
def test_either_side_of_the_ratio(more):
    """As many deletes as head slabs / 8, and one more: by the log, by the sweep."""
    say(f"case: compaction at the ratio, {more} more")
    n = 1 << 12
    v = np.arange(n)
    s = np.concatenate([v, v, v[: n // 2]])
    d = np.concatenate([(v + 1) % n, (v + 2) % n, (v[: n // 2] + 3) % n])
    p = Pair(n, s, d, np.ones(len(s), np.int64), views=native.VIEW_FWD)
    assert p.g.stats()["head_slabs"][0] == n
    k = n // 8 + more
    p.delete(s[:k], d[:k])
    assert p.g.compact() == 0  # one slab a chain: nothing to free, but every tombstone packed away
    p.check_structure()
    p.delete(s[k:3 * k:2], d[k:3 * k:2])
    p.g.compact()
    p.insert(s[:k], d[:k], np.ones(k, np.int64))
    p.check_structure()
    p.check_all(algos=("wcc",))


# without the undirected view: graphs on either side of the size from which the log is taken as with it,
# deletes on either side of its ratio there and of the one for smaller graphs
@pytest.mark.parametrize("views", [native.VIEW_FWD, native.VIEW_FWD | native.VIEW_REV])
@pytest.mark.parametrize("scale,share,more", [(16, 64, 0), (16, 64, 1), (20, 8, 0), (20, 8, 1)])
def test_ratios_without_the_undirected_view(views, scale, share, more):
    say(f"case: compaction, views {views}, scale {scale}, 1 delete in {share} head slabs, {more} more")
    g = I.rmat_graph(scale, 16, 31, device="cuda")
    graphs = [native.Graph(g.n, *g.u32(), views=views, log_capacity=k) for k in (0, 4096)]  # the second one sweeps
    heads = sum(graphs[0].stats()["head_slabs"])
    assert (heads >= 3 << 19) == (scale == 20)
    k = heads // share + more
    arcs = [x[:k].contiguous() for x in g.u32()]
    for _ in range(2):
        for G in graphs:
            for at in range(0, k, 4096 if G is graphs[1] else k):
                end = min(k, at + 4096) if G is graphs[1] else k
                G.delete_edges(arcs[0][at:end].contiguous(), arcs[1][at:end].contiguous())
        assert graphs[0].compact() == graphs[1].compact()
        assert graphs[0].stats()["pool_used"] == graphs[1].stats()["pool_used"]
        for G in graphs:
            assert G.compact() == 0
            assert G.check() == 0
            assert not bool(G.query_edges(arcs[0], arcs[1])[0].any())
            for at in range(0, k, 4096):
                G.insert_edges(*(x[at:at + 4096].contiguous() for x in arcs))
            assert G.check() == 0
            found, weight = G.query_edges(arcs[0], arcs[1])
            assert bool(found.all()) and torch.equal(weight, arcs[2])
        a, b = (sorted(zip(*(u32(x).tolist() for x in G.export()))) if scale < 20 else None for G in graphs)
        assert a == b
