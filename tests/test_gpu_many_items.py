"""Top-level passes over many items of small meshes: (top node, mesh) items in
one part, several at a time to a wave, whose survivors are counted together --
meshes of 1 to 97 triangles and empty ones, item counts around the rules' lines
(1,024 and 4,096), every pair and counter exactly the oracle's, plain, packed and
batched; and a bound on what so many items cost."""
import dataclasses

import numpy as np
import pytest

from conftest import workload
from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _cut(wl, sizes, seed):
    """The workload's first triangles as meshes of the given sizes."""
    rng = np.random.default_rng(seed)
    n = sum(sizes)
    at = rng.integers(0, wl.scene.m - n)
    tris = np.ascontiguousarray(wl.scene.tris[at:at + n])
    first = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.uint32)
    ball = np.zeros((len(sizes), 4), np.float32)
    for k, (a, c) in enumerate(zip(first, sizes)):
        if c:
            v = tris[a:a + c].reshape(-1, 3).astype(np.float64)
            mid = (0.5 * (v.min(0) + v.max(0))).astype(np.float32)
            ball[k] = [*mid, np.sqrt(((v - mid) ** 2).sum(1).max()) * 1.00001 + 1e-4]
    sc = dataclasses.replace(wl.scene, tris=tris, mesh_first=first, mesh_count=np.array(sizes, np.uint32),
                             mesh_sphere=ball, mesh_mat=np.zeros(len(sizes), np.int32))
    return dataclasses.replace(wl, scene=sc)


def _check(got, orc, pairs=True):
    t = orc["trav"]
    assert got["tests"] == t["tests"] and got["final_tests"] == t["final_tests"]
    assert (got["mesh_tests"], got["mesh_hits"]) == (t["mesh_tests"], t["mesh_hits"])
    if pairs:
        for lv, (a, b) in t["pairs"].items():
            assert np.array_equal(got["pairs"][lv][0], a) and np.array_equal(got["pairs"][lv][1], b), lv
    for a, b in zip(got["hit"], orc["hits"]):
        assert np.array_equal(np.asarray(a).view(np.uint32), np.asarray(b).view(np.uint32))


# pixels, B, levels, mesh sizes: 10 to 70,000 items
@pytest.mark.parametrize("w,h,B,n,sizes", [
    (16, 10, 8, 2, [97, 0]), (64, 16, 2, 2, [1, 63, 64, 65]), (64, 32, 4, 2, [3, 0, 90, 64]),
    (64, 32, 4, 2, [3, 0, 90, 64, 5]), (64, 48, 4, 2, [7, 1, 0, 65, 31] * 17), (64, 48, 2, 3, [1] * 300),
    (40, 30, 1, 1, [128, 2, 9] * 10)])
def test_many_small_items(w, h, B, n, sizes):
    import gpu_util
    wl = _cut(dataclasses.replace(workload("refl_1024", W=w, H=h), B=B, F=4, n=n), sizes, w + h)
    o = O.run_pipeline(wl)
    g = gpu_util.run_pipeline(wl)
    print(f"[many items] {g['mesh_tests']} items, {len(o['trav']['pairs'][n][0])} top-level pairs", flush=True)
    _check(g, o)
    _check(gpu_util.run_pipeline(wl, packed=True), o, pairs=False)


def test_many_small_items_batched():
    from paper_2312_06538_amd.batch import DeviceBatch
    base = dataclasses.replace(workload("refl_1024", W=64, H=48), B=4, F=4, n=2)
    wls = [_cut(base, s, k) for k, s in enumerate(([9, 0, 64] * 20, [70], [1, 2] * 50))]
    db = DeviceBatch(wls, 4, 4, 2, pair_capacity=1 << 20, keep_levels=True)
    m = db.run_with_retry()
    orcs = [O.run_pipeline(wl) for wl in wls]
    for f, (r, o) in enumerate(zip(db.frame_results(m), orcs)):
        print(f"[many items batched] frame {f}: {o['trav']['mesh_tests']} items", flush=True)
        for lv, (a, b) in o["trav"]["pairs"].items():
            assert np.array_equal(r["pairs"][lv][0], a) and np.array_equal(r["pairs"][lv][1], b), (f, lv)
    assert int(m.mesh_tests) == sum(o["trav"]["mesh_tests"] for o in orcs)
    assert int(m.tests[0]) == sum(o["trav"]["tests"][1] for o in orcs)


def test_many_small_items_cost():
    """The same leaves under 16 times the top nodes: 81,920 items of 256
    triangles on average took 2.4 times as long when they were cut in four,
    in one part 1.3 times."""
    from test_gpu_wide_levels import _traverse_us
    wl = workload("shadow_128", W=512, H=512)
    few, _ = _traverse_us(dataclasses.replace(wl, B=4, F=4, n=4))
    many, _ = _traverse_us(dataclasses.replace(wl, B=4, F=4, n=2))
    print(f"[many items] traversal {few:.0f} us under 1,024 top nodes, {many:.0f} us under 16,384", flush=True)
    assert many < 2.0 * few
