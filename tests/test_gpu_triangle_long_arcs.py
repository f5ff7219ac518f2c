"""Triangle updates whose batch edges join two vertices of many neighbours that are no hubs: walks
around the bucket counts at which a block takes over from a group, in a small and a large batch."""
import numpy as np
import pytest

from paper_2305_17813_amd import native
from parity import Pair, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("degree", [150, 175, 200, 640, 690, 1500])  # 15 .. 143 buckets
@pytest.mark.parametrize("extra", [0, 40_000])  # batch edges elsewhere: below and above 65,536 keys
def test_pairs_of_large_vertices(degree, extra):
    say(f"case: triangles, pairs of {degree} neighbours, {extra} edges elsewhere")
    rng = np.random.default_rng(degree + extra)
    n = 60_000
    big = np.arange(8)
    s = np.repeat(big, degree)
    d = np.concatenate([100 + rng.choice(3 * degree, degree, replace=False) for _ in big])
    p = Pair(n, s, d, np.ones(len(s), np.int64), views=native.VIEW_FWD | native.VIEW_UND, pool_slabs=200_000)
    p.check_tc()
    # an edge per pair (a vertex has too few batch edges to be a hub), and sparse edges elsewhere
    bs, bd = [big[0::2]], [big[1::2]]
    if extra:
        e = np.unique(np.sort(rng.integers(10_000, n, (extra, 2)), axis=1), axis=0)
        e = e[e[:, 0] != e[:, 1]]
        bs.append(e[:, 0])
        bd.append(e[:, 1])
    bs, bd = np.concatenate(bs), np.concatenate(bd)
    p.insert(bs, bd, np.ones(len(bs), np.int64))
    p.check_tc()
    p.delete(bs, bd)
    p.check_tc()
