"""Distance-only traversals, the paths that depend on sizes: steps that claim against steps that
mark and sweep, single-bucket chains against items of 16 buckets, frontiers of a few vertices
against several rows a lane, and the rounded distance bound over the whole range of distances."""
import numpy as np
import pytest
import torch

from paper_2305_17813_amd import inputs as I
from paper_2305_17813_amd import native

from parity import say

pytestmark = pytest.mark.gpu
INF = 0xFFFFFFFF


def reference(n, src, dst, w, source):
    """Levels by whole-edge-list relaxation, distances the same way with the saturating sum."""
    lv = np.full(n, INF, np.uint64)
    di = np.full(n, INF, np.uint64)
    lv[source] = di[source] = 0
    src, dst, w = src.astype(np.int64), dst.astype(np.int64), w.astype(np.uint64)
    for a, step in ((lv, np.ones_like(w)), (di, w)):
        while True:
            old = a.copy()
            m = a[src] != INF
            np.minimum.at(a, dst[m], np.minimum(a[src[m]] + step[m], INF - 1))
            if (a == old).all():
                break
    return lv.astype(np.uint32), di.astype(np.uint32)


def compare(n, src, dst, w, sources, **cfg):
    src, dst, w = (np.asarray(x, np.uint32) for x in (src, dst, w))
    t = [torch.from_numpy(x.view(np.int32).copy()).cuda() for x in (src, dst, w)]
    G = native.Graph(n, *t, views=native.VIEW_FWD | native.VIEW_REV, **cfg)
    for s in sources:
        lv, di = reference(n, src, dst, w, s)
        for kw in ({}, {"top_down_only": True}):
            got, _ = G.bfs_levels(s, **kw)
            assert np.array_equal(got.cpu().numpy().view(np.uint32), lv), (s, kw)
        assert np.array_equal(G.sssp_distances(s).cpu().numpy().view(np.uint32), di), s


def arcs(rng, n, m, weights):
    key = np.unique(rng.integers(0, n * n, m, dtype=np.int64))
    rng.shuffle(key)
    src, dst = key // n, key % n
    keep = src != dst
    return src[keep], dst[keep], weights(keep.sum())


# one vertex short of, exactly at and past a wave, a block and a row of them; a hub of several
# items of 16 buckets whose arcs reach every vertex
@pytest.mark.parametrize("n", [1, 2, 15, 17, 63, 64, 65, 255, 257, 4099])
@pytest.mark.parametrize("delta", [0, 7])
def test_hub_and_ring(n, delta):
    say(f"case: hub and ring, {n} vertices, band {delta}")
    v = np.arange(n)
    ring = v if n > 1 else v[:0]
    hub = v[1:]
    src = np.concatenate([ring, np.zeros(len(hub), np.int64)])
    dst = np.concatenate([(ring + 1) % max(n, 1), hub])
    key, first = np.unique(src * n + dst, return_index=True)
    w = (np.arange(len(src)) * 2654435761 % 97 + 1).astype(np.uint32)
    compare(n, src[first], dst[first], w[first], sorted({0, n // 2, n - 1}), sssp_delta=delta)


# weights from one to the saturation of the sums: every exponent of the rounded bound
@pytest.mark.parametrize("bits", [1, 3, 4, 5, 9, 16, 24, 31, 32])
def test_weight_ranges(bits):
    say(f"case: weights of up to {bits} bits")
    rng = np.random.default_rng(100 + bits)
    hi = (1 << bits) - 1
    weights = lambda k: np.maximum(1, rng.integers(max(1, hi // 3), hi + 1, k)).astype(np.uint32)
    src, dst, w = arcs(rng, 700, 4000, weights)
    compare(700, src, dst, w, [int(src[0]), 3])
    compare(700, src, dst, w, [5], sssp_delta=max(1, hi // 2))


# power-law graphs: dense steps, many repeated relaxations of the same vertices
@pytest.mark.parametrize("scale,ef", [(9, 16), (13, 8), (14, 4)])
def test_power_law(scale, ef):
    say(f"case: power-law graph, scale {scale}, edge factor {ef}")
    g = I.rmat_graph(scale, ef, 7 + scale)
    a = [np.asarray(x.cpu()).view(np.uint32) if torch.is_tensor(x) else np.asarray(x) for x in g.u32()]
    deg = np.bincount(a[0].astype(np.int64), minlength=g.n)
    compare(g.n, *a, [int(deg.argmax()), int(np.nonzero(deg == 1)[0][0])])


# bands of a fraction of a weight on a graph of many blocks: many splits, of piles that most blocks
# have a share in
@pytest.mark.parametrize("scale,ef,delta", [(16, 8, 3), (17, 4, 20), (18, 8, 200)])
def test_many_splits_of_large_piles(scale, ef, delta, orc):
    say(f"case: far-pile splits, scale {scale}, edge factor {ef}, band {delta}")
    g = I.rmat_graph(scale, ef, 3)
    s, d, w = (np.asarray(x.cpu()).view(np.uint32) for x in g.u32())
    O = orc.OracleGraph(g.n, s, d, w)
    G = native.Graph(g.n, *g.u32(), views=native.VIEW_FWD | native.VIEW_REV, sssp_delta=delta)
    for u in (int(np.bincount(s).argmax()), int(s[len(s) // 2])):
        want, parent = O.sssp(u)
        ws = torch.empty(native.load().mk_sssp_distances_workspace_bytes(G.h), dtype=torch.uint8, device="cuda")
        for _ in range(3):
            assert np.array_equal(G.sssp_distances(u, ws=ws).cpu().numpy().view(np.uint32), want)
        di, pa = G.sssp(u, mode=native.RECOMPUTE)
        assert np.array_equal(di.cpu().numpy().view(np.uint32), want)
        assert np.array_equal(pa.cpu().numpy().view(np.uint32), parent)


@pytest.mark.parametrize("n", [1, 63, 257, 5000])
def test_workspaces_fit_where_they_did(n):
    """The sizes that programs may have noted down: two queues of n words for the levels, six arrays of
    n words for the distances, and the work items."""
    say(f"case: workspace sizes, {n} vertices")
    rng = np.random.default_rng(n)
    src, dst, w = arcs(rng, n, 40 * n, lambda k: rng.integers(1, 90, k))
    G = native.Graph(n, src, dst, w, views=native.VIEW_FWD | native.VIEW_REV)
    items = 2 * ((n + G.stats()["head_slabs"][0] // 16 + 64) * 4 + 256)
    lib = native.load()
    lv_bytes, di_bytes = 256 + 2 * (4 * n + 256) + items + 256, 256 + 6 * (4 * n + 256) + items + 256
    assert lib.mk_bfs_levels_workspace_bytes(G.h) <= lv_bytes
    assert lib.mk_sssp_distances_workspace_bytes(G.h) <= di_bytes
    lv, di = reference(n, np.asarray(src, np.uint32), np.asarray(dst, np.uint32), np.asarray(w, np.uint32), 0)
    # the workspace ends where the last of the needed bytes does, and what lies behind it stays as it was
    for need, call, want in ((lib.mk_bfs_levels_workspace_bytes(G.h), lambda ws: G.bfs_levels(0, ws=ws)[0], lv),
                             (lib.mk_sssp_distances_workspace_bytes(G.h), lambda ws: G.sssp_distances(0, ws=ws), di)):
        room = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        got = call(room[:need])
        assert np.array_equal(got.cpu().numpy().view(np.uint32), want)
        assert bool((room[need:] == 0xA5).all())


# no vertex with several buckets: no work items, one launch less a step; long chains, rows of vertices a
# lane, and a frontier of one vertex for many steps
@pytest.mark.parametrize("name,load_factor", [("power law", 0.0), ("wide", 0.0), ("wide", 0.7), ("grid", 0.7)])
def test_single_bucket_graphs(name, load_factor):
    say(f"case: distances on single-bucket graphs, {name}, load factor {load_factor}")
    rng = np.random.default_rng(5)
    if name == "grid":
        g = I.grid_graph(60, 3)
        src, dst, w = (np.asarray(x.cpu()).view(np.uint32) for x in g.u32())
        n = g.n
    elif name == "power law":
        g = I.rmat_graph(11, 8, 3)
        src, dst, w = (np.asarray(x.cpu()).view(np.uint32) for x in g.u32())
        n = g.n
    else:  # 0 -> 300 -> 90,000 -> 90,000, three arcs a vertex at most
        n = 1 + 300 + 180_000
        a = 301 + np.arange(90_000)
        src = np.concatenate([np.zeros(300, np.int64), 1 + np.arange(90_000) % 300, a, a])
        dst = np.concatenate([1 + np.arange(300), a, 90_000 + rng.permutation(a), 90_000 + rng.permutation(a)])
        key = np.unique(src * n + dst)
        src, dst = key // n, key % n
        w = rng.integers(1, 40, len(src))
        if load_factor:  # the first vertices' arcs fill several buckets: only the rest as a graph of its own
            keep = src > 300
            src, dst, w = src[keep] - 301, dst[keep] - 301, w[keep]
            n -= 301
    w = np.asarray(w, np.uint32)
    G = native.Graph(n, np.asarray(src, np.int64), np.asarray(dst, np.int64), w.astype(np.int64),
                     views=native.VIEW_FWD, load_factor=load_factor)
    assert G.stats()["head_slabs"][0] == n
    G.close()
    compare(n, src, dst, w, [int(src[0]), int(src[-1])], load_factor=load_factor)


# top-down alone, large and dense enough to mark and sweep, and one vertex or a few arcs short of that
@pytest.mark.parametrize("n,m", [(1 << 20, 9 << 20), ((1 << 20) - 1, 9 << 20), (1 << 20, 7 << 20), (3001, 24 * 3001),
                                 (3001, 24 * 3001 - 1)])
def test_top_down_alone(n, m, orc):
    say(f"case: levels top down, {n} vertices, {m} arcs")
    g = I.er_graph(n, m, 3)
    want, _ = orc.OracleGraph(n, *(np.asarray(x.cpu()).view(np.uint32) for x in g.u32())).bfs(5)
    for views in (native.VIEW_FWD, native.VIEW_FWD | native.VIEW_REV):
        G = native.Graph(n, *g.u32(), views=views)
        for _ in range(2):
            assert np.array_equal(G.bfs_levels(5, top_down_only=True)[0].cpu().numpy().view(np.uint32), want)
        G.close()
