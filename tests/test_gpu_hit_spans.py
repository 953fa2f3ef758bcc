"""Final tests of chunks whose pairs lie in leaves far apart -- more leaves
between the first and the last than there are bins, so that only the leaves that
have pairs get one -- or in few leaves, which get many bins each: at both sides
of the number of bins, of the span that a round covers and of a chunk, stored,
packed, fused and batched; every hit and counter exactly the oracle's.  And
bounds on what such chunks cost."""
import dataclasses

import numpy as np
import pytest

from conftest import workload
from oracle import oracle as O

pytestmark = pytest.mark.gpu

BINS, SPAN = 1024, 32768


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _scene(rng, n, m):
    from workloads.scenes import Scene
    v0 = rng.uniform(-10, 10, (m, 3))
    tris = np.stack([v0, v0 + rng.normal(0, 3, (m, 3)), v0 + rng.normal(0, 3, (m, 3))], 1).astype(np.float32)
    o = rng.uniform(-20, 20, (n, 3))
    d = tris[rng.integers(0, m, n)].mean(1) - o
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    sc = Scene(tris=tris, mesh_first=np.zeros(1, np.uint32), mesh_count=np.array([m], np.uint32),
               mesh_sphere=np.array([[0, 0, 0, 1e30]], np.float32), mesh_mat=np.zeros(1, np.int32),
               mat_flags=np.zeros(1, np.uint32), mat_ior=np.ones(1, np.float32))
    o, d = o.astype(np.float32), d.astype(np.float32)
    rays = {"ox": o[:, 0], "oy": o[:, 1], "oz": o[:, 2], "dx": d[:, 0], "dy": d[:, 1], "dz": d[:, 2],
            "tmax": np.full(n, np.finfo(np.float32).max, np.float32), "pix": np.zeros(n, np.uint32)}
    return sc, rays


# B, leaves, leaves that have pairs, pairs (64 to a chunk up to 80,000; above
# 5.3 M a chunk holds the most, 4,096)
@pytest.mark.parametrize("B,leaves,used,n_pairs", [
    (4, BINS - 1, 60, 5000), (4, BINS, 60, 5000), (4, BINS + 1, 64, 5001), (16, 20000, 3000, 60000),
    (3, SPAN, 200, 70000), (2, SPAN + 1, 200, 70000), (1, 3 * SPAN + 77, 5000, 70000), (32, 1500, 1500, 40000),
    (8, SPAN - 1, 30000, 70000), (4, 5000, BINS, 5500000), (4, 5000, BINS + 1, 5500000),
    (2, 2 * SPAN + 3, 40000, 5500000), (1, 4097, 4097, 5500001)])
def test_spread_leaves_match_oracle(B, leaves, used, n_pairs):
    import gpu_util
    rng = np.random.default_rng(B + leaves)
    n = leaves * B - (B > 1)                # the last leaf is not whole
    sc, rays = _scene(rng, n, 97)
    some = np.sort(rng.choice(leaves, used, replace=False))
    some[0], some[-1] = 0, leaves - 1       # the whole span in most chunks
    node = some[rng.integers(0, used, n_pairs)]
    ends = rng.random(n_pairs) < 0.05
    node[ends] = some[rng.integers(0, 2, int(ends.sum())) * (used - 1)]
    pairs = rng.integers(0, 97, n_pairs).astype(np.uint32), node.astype(np.uint32)
    ids = rng.permutation(n).astype(np.uint32)
    print(f"[hit spans] B={B} {used} of {leaves} leaves, {n_pairs} pairs", flush=True)
    stages = {}
    ref = O.closest_hit(rays, ids, B, pairs, sc, 1e-4, stages=stages)
    g, meta = gpu_util.gpu_closest_hit(rays, ids, B, pairs, sc, 1e-4)
    for a, b in zip(g, ref):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    assert int(meta.final_tests) == int(np.minimum(B, n - pairs[1].astype(np.int64) * B).sum())
    assert (int(meta.final_u_pass), int(meta.final_uv_pass)) == (stages["u"], stages["uv"])


# leaves in all, those that have pairs; `most`: the share of the pairs in one of them
@pytest.mark.parametrize("B,leaves,used,most,n_pairs", [
    (16, 40, 1, 0.0, 9000), (4, 1, 1, 0.0, 5500001), (4, 5, 4, 0.0, 5500000), (2, 5, 5, 0.9, 5500000),
    (8, 17, 16, 0.0, 5500000), (16, 17, 17, 0.5, 5500000), (1, 70, 64, 0.0, 5400000), (3, 256, 255, 0.99, 5500000),
    (32, 256, 256, 0.0, 1400000), (4, 257, 257, 0.5, 5500000), (4, 9000, 200, 0.3, 5500000), (4, 40000, 3, 0.0, 70000)])
def test_few_leaves_match_oracle(B, leaves, used, most, n_pairs):
    import gpu_util
    rng = np.random.default_rng(B + leaves)
    n = leaves * B - (B > 1)
    sc, rays = _scene(rng, n, 97)
    some = np.sort(rng.choice(leaves, used, replace=False))
    some[-1] = leaves - 1
    node = np.where(rng.random(n_pairs) < most, some[used // 2], some[rng.integers(0, used, n_pairs)])
    pairs = rng.integers(0, 97, n_pairs).astype(np.uint32), node.astype(np.uint32)
    ids = rng.permutation(n).astype(np.uint32)
    print(f"[hit few] B={B} {used} of {leaves} leaves, {n_pairs} pairs", flush=True)
    stages = {}
    ref = O.closest_hit(rays, ids, B, pairs, sc, 1e-4, stages=stages)
    g, meta = gpu_util.gpu_closest_hit(rays, ids, B, pairs, sc, 1e-4)
    for a, b in zip(g, ref):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    assert int(meta.final_tests) == int(np.minimum(B, n - pairs[1].astype(np.int64) * B).sum())
    assert (int(meta.final_u_pass), int(meta.final_uv_pass)) == (stages["u"], stages["uv"])


@pytest.mark.parametrize("B,F,n", [(4, 4, 1), (8, 4, 2), (2, 2, 3), (32, 8, 2)])
def test_flat_hierarchies_match_oracle(B, F, n):
    test_wide_hierarchies_match_oracle(B, F, n)


@pytest.mark.parametrize("B,F,n", [(4, 4, 7), (2, 4, 8), (2, 16, 4), (8, 2, 12), (1, 8, 6)])
def test_wide_hierarchies_match_oracle(B, F, n):
    import gpu_util
    from paper_2312_06538_amd.batch import DeviceBatch
    wls = [dataclasses.replace(workload("mixed_1080p", W=w, H=h, n_meshes=24), B=B, F=F, n=n)
           for w, h in ((96, 60), (40, 30))]
    orcs = [O.run_pipeline(wl) for wl in wls]
    t = orcs[0]["trav"]
    print(f"[hit spans] B={B} F={F} n={n}: {len(t['pairs'][1][0])} level-1 pairs", flush=True)
    for kw in ({}, {"leaf_hit": True}, {"packed": True}):
        g = gpu_util.run_pipeline(wls[0], keep_levels=False, **kw)
        assert g["final_tests"] == t["final_tests"], kw
        for a, b in zip(g["hit"], orcs[0]["hits"]):
            assert np.array_equal(np.asarray(a).view(np.uint32), np.asarray(b).view(np.uint32)), kw
    for fused in (False, True):
        db = DeviceBatch(wls, B, F, n, pair_capacity=1 << 20, leaf_hit=fused)
        m = db.run_with_retry()
        assert int(m.final_tests) == sum(o["trav"]["final_tests"] for o in orcs)
        for r, o in zip(db.frame_results(m, with_pairs=False), orcs):
            for a, b in zip(r["hit"], o["hits"]):
                assert np.array_equal(np.asarray(a).view(np.uint32), np.asarray(b).view(np.uint32)), fused


def _hit_us(leaves, stride, idx, tri, B=4, tmax=None):
    """Final tests of the pairs (tri[i], leaf idx[i] * stride)."""
    import gpu_util
    import torch
    from paper_2312_06538_amd import crsh as X
    n = leaves * stride * B
    sc, rays = _scene(np.random.default_rng(1), n, 500)
    if tmax is not None:
        rays["tmax"][:] = tmax
    r = {k: gpu_util.dev_f32(rays[k]) for k in gpu_util.RAY_KEYS}
    c_r = X.Rays(*[r[k].data_ptr() for k in gpu_util.RAY_KEYS], None, n)
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    node = (idx * stride).to(torch.int32)
    pairs = X.Pairs(tri.data_ptr(), node.data_ptr(), len(idx))
    c_sc, keep = gpu_util._scene(sc)
    out = [torch.zeros(n, dtype=dt, device="cuda") for dt in (torch.int64, torch.int32, *[torch.float32] * 3)]
    hits = X.Hits(*[x.data_ptr() for x in out], n)
    meta = gpu_util.new_meta(n_rays=n, n_levels=1, pairs=[len(idx)])
    wsb = X.crsh_workspace_size(n, sc.m, 1, 1, 1)
    ws = gpu_util.ws_tensor(wsb)
    best = float("inf")
    for _ in range(6):
        X.crsh_hits_reset(hits, gpu_util.s())
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        X.crsh_closest_hit(c_r, ids.data_ptr(), B, pairs, c_sc, 1e-4, hits, meta.data_ptr(), ws.data_ptr(), wsb,
                           gpu_util.s())
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


def test_spread_leaves_cost():
    """The same pairs in 256 leaves side by side and 64 apart: taken window by
    window the second are read 16 times, by the leaves that have pairs once (and
    once more for their bitmap)."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(3)
    k = 16 << 20
    idx = torch.randint(0, 256, (k,), device="cuda", generator=gen)
    tri = torch.randint(0, 500, (k,), device="cuda", generator=gen, dtype=torch.int32)
    near, far = _hit_us(256, 1, idx, tri), _hit_us(256, 64, idx, tri)
    print(f"[hit spans] {near:.0f} us side by side, {far:.0f} us spread", flush=True)
    assert far < 1.7 * near


def test_few_leaves_cost():
    """Pairs of 4 leaves and of 512, with no hits (their minima would meet at the
    few rays): 1.7 times as long with one bin a leaf, no longer with 256 each."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(4)
    k = 16 << 20
    idx = torch.randint(0, 512, (k,), device="cuda", generator=gen)
    tri = torch.randint(0, 500, (k,), device="cuda", generator=gen, dtype=torch.int32)
    many, few = _hit_us(512, 1, idx, tri, tmax=0.0), _hit_us(4, 1, idx // 128, tri, tmax=0.0)
    print(f"[hit few] {many:.0f} us in 512 leaves, {few:.0f} us in 4", flush=True)
    assert few < 1.6 * many
