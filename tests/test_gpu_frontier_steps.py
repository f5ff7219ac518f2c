"""Frontier kernels at the sizes where one block goes on by itself: frontiers around the 512
vertices it starts with and the 1,024 it can stage, depths around the 64 steps of one launch, and
vertices with many buckets (more than a block collects) in such a frontier."""
import time

import numpy as np
import pytest
import torch

from paper_2305_17813_amd import native
from parity import Pair, say

pytestmark = pytest.mark.gpu

VIEWS = native.VIEW_FWD | native.VIEW_REV


def broom(width, depth):
    """0 -> `width` paths of `depth` vertices each; weights vary so that SSSP re-relaxes."""
    rng = np.random.default_rng(width * 1000 + depth)
    first = 1 + np.arange(width) * depth
    s = [np.zeros(width, np.int64)] + [first + k for k in range(depth - 1)]
    d = [first] + [first + k + 1 for k in range(depth - 1)]
    s, d = np.concatenate(s), np.concatenate(d)
    return s, d, rng.integers(1, 50, len(s)), 1 + width * depth


def layers(width, count, fan):
    """`count` layers of `width` vertices, `fan` random arcs from each into the next layer."""
    rng = np.random.default_rng(width + 7 * count + fan)
    s, d = [np.zeros(width, np.int64)], [1 + np.arange(width)]
    for k in range(count - 1):
        base = 1 + k * width
        for v in range(width):
            t = rng.choice(width, size=min(fan, width), replace=False)
            s.append(np.full(len(t), base + v))
            d.append(base + width + t)
    s, d = np.concatenate(s), np.concatenate(d)
    return s, d, rng.integers(1, 30, len(s)), 1 + width * count


CASES = {
    "paths of 63": broom(3, 63), "paths of 64": broom(3, 64), "paths of 65": broom(3, 65),
    "paths of 200": broom(2, 200),
    "511 wide": broom(511, 5), "512 wide": broom(512, 5), "513 wide": broom(513, 5),
    "1024 wide": broom(1024, 4), "1025 wide": broom(1025, 4),
    "layers, one bucket": layers(300, 6, 4),
    "layers, several buckets": layers(120, 6, 100),  # up to 10 buckets each: over 1,024 chains
    "layers, heavy": layers(250, 4, 240),  # 23 buckets each
}


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("views", [VIEWS, native.VIEW_FWD])
def test_inserts_and_deletes_through_small_frontiers(name, views):
    say(f"case: frontier steps, {name}, views {views}")
    s, d, w, n = CASES[name]
    # a graph of its own vertices first, so that each batch is a small frontier with a long tail
    p = Pair(n, s, d, w, views=views, sssp_delta=40)
    p.check_all(algos=("bfs", "sssp"))
    cut = np.nonzero(s == 0)[0][::2]  # half of the source's arcs: whole subtrees are invalidated
    for _ in range(2):
        p.delete(s[cut], d[cut])
        p.check_all(algos=("bfs", "sssp"))
        p.insert(s[cut], d[cut], w[cut])
        p.check_all(algos=("bfs", "sssp"))
    p.check_all(mode=native.RECOMPUTE, algos=("bfs", "sssp"))
    ws = p.g.traversal_workspace()
    for weighted, want in ((False, p.o.bfs(0)), (True, p.o.sssp(0))):
        di, pa = p.g.traverse_from(0, weighted, ws)
        assert np.array_equal(di.cpu().numpy().view(np.uint32), want[0])
        assert np.array_equal(pa.cpu().numpy().view(np.uint32), want[1])


def rare_fans(width, every, fan, layers):
    """`layers` layers of `width` vertices: each vertex has one arc into the next layer, every
    `every`-th one `fan` more (several buckets among many single ones)."""
    rng = np.random.default_rng(width + every + fan)
    s, d = [np.zeros(width, np.int64)], [1 + np.arange(width)]
    for k in range(layers - 1):
        base = 1 + k * width
        s.append(base + np.arange(width))
        d.append(base + width + rng.permutation(width))
        big = base + np.arange(0, width, every)
        s.append(np.repeat(big, fan))
        d.append(base + width + rng.integers(0, width, len(big) * fan))
    s, d = np.concatenate(s), np.concatenate(d)
    key = np.unique(s * (2 * width * layers) + d)
    s, d = key // (2 * width * layers), key % (2 * width * layers)
    return s, d, rng.integers(1, 30, len(s)), 1 + width * layers


# several rounds of 256 vertices in one block, of which some collect further buckets and some do
# not: inner frontiers of up to 1,024 vertices, and frontiers of more rounds than there are blocks
@pytest.mark.parametrize("width,every,fan,layers", [(257, 256, 30, 5), (512, 300, 150, 5), (900, 400, 100, 4),
                                                    (1024, 1, 20, 4), (1024, 511, 160, 4), (700_000, 5000, 120, 2)])
def test_rounds_with_and_without_further_buckets(width, every, fan, layers):
    say(f"case: frontier rounds, {width} wide, {fan} more arcs every {every}")
    s, d, w, n = rare_fans(width, every, fan, layers)
    p = Pair(n, s, d, w, views=VIEWS, sssp_delta=25)
    p.check_all(algos=("bfs", "sssp"))
    cut = np.nonzero(s == 0)[0]
    for part in (cut, cut[::3], cut[:300]):
        p.delete(s[part], d[part])
        p.check_all(algos=("bfs", "sssp"))
        p.insert(s[part], d[part], w[part])
        p.check_all(algos=("bfs", "sssp"))


def even_layers(width, fan, layers):
    """`layers` layers; every vertex has about `fan` arcs into the next one."""
    rng = np.random.default_rng(width * 31 + fan)
    s, d = [np.zeros(width, np.int64)], [1 + np.arange(width)]
    for k in range(layers - 1):
        base = 1 + k * width
        s.append(np.repeat(base + np.arange(width), fan))
        d.append(base + width + rng.integers(0, width, width * fan))
    s, d = np.concatenate(s), np.concatenate(d)
    n = 1 + width * layers
    key = np.unique(s * n + d)
    return key // n, key % n, rng.integers(1, 60, len(key)), n


# how a launch's blocks share the light vertices: 256 buckets in one block and one more, 384 and 512
# where there are two a vertex; 16 lanes a vertex where there are many buckets on average (fans of 60 and 150) and up to 16,384 vertices; beyond
# that blocks of 32 to 256 vertices (fan 14, two buckets each, one bucket under a larger load factor)
@pytest.mark.parametrize("width,fan,layers", [(31, 80, 5), (32, 80, 4), (33, 80, 4), (128, 20, 4), (129, 20, 4),
                                              (192, 14, 4), (193, 14, 4), (256, 14, 5), (257, 14, 5),
                                              (2000, 60, 4), (6000, 150, 3), (16_384, 14, 3), (16_385, 14, 3),
                                              (60_000, 14, 3)])
@pytest.mark.parametrize("load_factor", [0.7, 3.0])
def test_shares_of_the_blocks(width, fan, layers, load_factor):
    say(f"case: frontier shares, {width} wide, fan {fan}, load factor {load_factor}")
    s, d, w, n = even_layers(width, fan, layers)
    p = Pair(n, s, d, w, views=VIEWS, sssp_delta=20, load_factor=load_factor)
    p.check_all(algos=("bfs", "sssp"))
    cut = np.nonzero(s == 0)[0]
    for part in (cut, cut[::2]):
        p.delete(s[part], d[part])
        p.check_all(algos=("bfs", "sssp"))
        p.insert(s[part], d[part], w[part])
        p.check_all(algos=("bfs", "sssp"))
    ws = p.g.traversal_workspace()
    for weighted, want in ((False, p.o.bfs(0)), (True, p.o.sssp(0))):
        di, pa = p.g.traverse_from(0, weighted, ws)
        assert np.array_equal(di.cpu().numpy().view(np.uint32), want[0])
        assert np.array_equal(pa.cpu().numpy().view(np.uint32), want[1])


def test_dense_graph_fills_the_chip():
    """20,000 vertices of 15 buckets: far more lanes than one block's share of 256 vertices keeps
    busy.  Against the levels of the same graph, whose kernels share the slabs differently."""
    say("case: traversal of a dense graph, time")
    rng = np.random.default_rng(2)
    key = np.unique(rng.integers(0, 20_000 ** 2, 3_000_000))
    s, d = key // 20_000, key % 20_000
    g = native.Graph(20_000, s, d, views=VIEWS)
    ws = g.traversal_workspace()

    def fastest(call):
        us = []
        for _ in range(9):
            torch.cuda.synchronize()
            t = time.perf_counter()
            call()
            torch.cuda.synchronize()
            us.append(time.perf_counter() - t)
        return min(us)

    # 245 us against 126 top down; it was 560
    assert fastest(lambda: g.traverse_from(0, False, ws)) <= 3.2 * fastest(lambda: g.bfs_levels(0, top_down_only=True))
