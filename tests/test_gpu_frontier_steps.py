"""Frontier kernels at the sizes where one block goes on by itself: frontiers around the 512
vertices it starts with and the 1,024 it can stage, depths around the 64 steps of one launch, and
vertices with many buckets (more than a block collects) in such a frontier."""
import numpy as np
import pytest

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
