"""Traversal levels at the edges of the level step's tiles (512 or 1,024
parent pairs): top-level pair counts just below, at and above whole tiles, for
merge factors on both sides of every mask and tile width, and storage that ends
inside a tile -- every level bit-exact against the oracle, or its exact prefix
where the storage ends."""
import numpy as np
import pytest

from conftest import oracle_run, small, workload
from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _tree(B, F, n):
    base, kw = small("refl_96")
    wl = workload(base, **kw)
    o = oracle_run(base, **kw)
    return wl, O.build_tree(o["hash"]["rays"], o["sorted_ids"], B, F, n)


def _end_for(tree, sc, want):
    """The fewest triangles from the first on with at least `want` top-level pairs."""
    top = tree["n_levels"]
    lo, hi = 1, 64
    count = lambda e: len(O.traverse(tree, sc, 0, e)["pairs"][top][0])
    while hi < sc.m and count(hi) < want:
        lo, hi = hi, min(2 * hi, sc.m)
    while lo < hi:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if count(mid) >= want else (mid + 1, hi)
    return lo


@pytest.mark.parametrize("B,F,n", [(16, 4, 4), (8, 3, 4), (16, 8, 3), (4, 5, 4), (16, 16, 3), (16, 2, 6)])
@pytest.mark.parametrize("want", [1, 511, 1024, 1025])
def test_levels_at_tile_edges(B, F, n, want):
    import gpu_util
    wl, tree = _tree(B, F, n)
    e = _end_for(tree, wl.scene, want)
    ot = O.traverse(tree, wl.scene, 0, e)
    print(f"[level step] B={B} F={F} n={n}: {[len(t) for t, _ in ot['pairs'].values()]} pairs", flush=True)
    cap = max(len(t) for t, _ in ot["pairs"].values()) + 1
    g = gpu_util.gpu_traverse(tree, wl.scene, B, F, batches=[(0, e)], capacity=cap)
    assert g["status"] == 0
    for lv, (t, nd) in ot["pairs"].items():
        assert np.array_equal(g["pairs"][lv][0], t) and np.array_equal(g["pairs"][lv][1], nd), lv
        assert g["tests"][lv] == ot["tests"][lv] and g["hits"][lv] == ot["hits"][lv], lv


@pytest.mark.parametrize("F,cap", [(4, 1), (4, 1000), (4, 1537), (8, 513), (16, 4097)])
def test_storage_that_ends_inside_a_tile(F, cap):
    """Each level holds the first `cap` of the pairs that the level above's
    stored pairs lead to, in order."""
    import gpu_util
    wl, tree = _tree(16, F, 3)
    ot = O.traverse(tree, wl.scene, 0, wl.scene.m)
    g = gpu_util.gpu_traverse(tree, wl.scene, 16, F, capacity=cap)
    assert g["status"] == 2
    top = tree["n_levels"]
    assert int(g["meta"].pairs[top - 1]) == len(ot["pairs"][top][0])
    key = lambda t, nd: t.astype(np.int64) << 32 | nd.astype(np.int64)
    for lv in range(top, 0, -1):
        t, nd = ot["pairs"][lv]
        k = len(t)
        if lv < top:    # the children of the parents that were stored
            pt, pn = ot["pairs"][lv + 1]
            pt, pn = pt[:stored], pn[:stored]
            k = int(np.isin(key(t, nd // F), key(pt, pn)).sum())
            cnt = int(tree["level_cnt"][lv - 1])
            assert g["tests"][lv] == int(np.minimum(F, cnt - pn.astype(np.int64) * F).sum())
        assert g["hits"][lv] == k
        stored = min(k, cap)
        assert np.array_equal(g["pairs"][lv][0], t[:stored]) and np.array_equal(g["pairs"][lv][1], nd[:stored]), lv
