"""The final tests' matrix filter against the oracle, where it can go wrong:
every group width and the bundles at its edges, chunks and leaf windows that
are not whole, rays aimed at edges and vertices (u at 0 and 1), and lengths
outside the filter's range (zero, tiny, huge, infinite, NaN).  The filter only
decides which tests are made in full, so every result and counter is exact:
triangle ids, bits of t, u, v, and the u and u-v passes."""
import numpy as np
import pytest

from oracle import oracle as O
from workloads.scenes import Scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _case(seed, n, m, n_pairs, B, scale, odd):
    """n rays, m triangles and n_pairs (triangle, leaf) pairs in runs of
    neighbouring leaves; `odd`: a tenth of the rays and triangles special."""
    rng = np.random.default_rng(seed)
    v0 = rng.uniform(-10, 10, (m, 3)) * scale
    tris = np.stack([v0, v0 + rng.normal(0, 1, (m, 3)) * scale, v0 + rng.normal(0, 1, (m, 3)) * scale], 1)
    o = rng.uniform(-20, 20, (n, 3)) * scale
    # towards a point of a triangle's plane: inside, on an edge, at a vertex
    # or beyond, at equal shares
    k = rng.integers(0, m, n)
    w = rng.uniform(0, 1, (n, 2))
    w[w.sum(1) > 1] = 1 - w[w.sum(1) > 1]
    kind = rng.integers(0, 5, n)
    w[kind == 1, 0] = 0.0
    w[kind == 2, 0] = 1.0 - w[kind == 2, 1]
    w[kind == 3] = rng.integers(0, 2, (int((kind == 3).sum()), 2))
    w[kind == 4] = rng.uniform(-3, 3, (int((kind == 4).sum()), 2))
    p = tris[k, 0] + w[:, :1] * (tris[k, 1] - tris[k, 0]) + w[:, 1:] * (tris[k, 2] - tris[k, 0])
    d = p - o
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    o, d, tris = o.astype(np.float32), d.astype(np.float32), tris.astype(np.float32)
    tmax = np.where(rng.uniform(size=n) < 0.5, np.finfo(np.float32).max, 15.0 * scale).astype(np.float32)
    if odd:
        for i in rng.choice(n, n // 10, replace=False):
            f = [0.0, 1e-4, 1e7, 1e25, 1e-30, np.inf, np.nan, -0.0][int(rng.integers(0, 8))]
            with np.errstate(all="ignore"):
                [o, d][int(rng.integers(0, 2))][i] *= np.float32(f)
        for i in rng.choice(m, m // 10, replace=False):
            c = int(rng.integers(0, 5))
            with np.errstate(all="ignore"):
                if c == 0:
                    tris[i, 2] = tris[i, 1]
                elif c == 1:
                    tris[i, 1:] = tris[i, 0]
                else:
                    tris[i] *= np.float32([1e8, 1e20, 1e-25][c - 2])
    leaves = -(-n // B)
    run = rng.integers(0, leaves, -(-n_pairs // 7))
    node = np.minimum(run[:, None] + np.arange(7)[None, :], leaves - 1).reshape(-1)[:n_pairs]
    tri = np.repeat(rng.integers(0, m, len(run)), 7)[:n_pairs]
    sc = Scene(tris=tris, mesh_first=np.zeros(1, np.uint32), mesh_count=np.array([m], np.uint32),
               mesh_sphere=np.array([[0, 0, 0, 1e30]], np.float32), mesh_mat=np.zeros(1, np.int32),
               mat_flags=np.zeros(1, np.uint32), mat_ior=np.ones(1, np.float32))
    rays = {"ox": o[:, 0], "oy": o[:, 1], "oz": o[:, 2], "dx": d[:, 0], "dy": d[:, 1], "dz": d[:, 2], "tmax": tmax,
            "pix": np.zeros(n, np.uint32)}
    return sc, rays, rng.permutation(n).astype(np.uint32), (tri.astype(np.uint32), node.astype(np.uint32))


# B, rays, triangles, pairs, scale, special values.  Chunks hold 256 to 4,096
# pairs and a window 1,024 leaves: one pair, one short of and one past a
# chunk, and 40,000 pairs over up to 6,000 leaves (several windows per chunk)
@pytest.mark.parametrize("B,n,m,n_pairs,scale,odd", [
    (1, 700, 50, 9000, 1.0, False), (3, 1000, 300, 4097, 1.0, True), (4, 4096, 33, 257, 1.0, False),
    (5, 3001, 100, 20000, 1.0, True), (8, 48000, 500, 40000, 1.0, False), (9, 2000, 64, 255, 1.0, False),
    (13, 40, 7, 1, 1.0, False), (16, 5000, 1000, 300001, 1.0, True), (16, 33, 5, 4096, 1e-3, False),
    (16, 2000, 200, 30000, 1e3, True), (17, 3000, 200, 30000, 1.0, False), (31, 31, 40, 64, 1.0, True),
    (32, 6000, 200, 50000, 1.0, True)])
def test_filtered_final_tests_match_oracle(B, n, m, n_pairs, scale, odd):
    import gpu_util
    print(f"[hit filter] B={B} rays={n} triangles={m} pairs={n_pairs} scale={scale} odd={odd}", flush=True)
    sc, rays, ids, pairs = _case(B + n, n, m, n_pairs, B, scale, odd)
    stages = {}
    ref = O.closest_hit(rays, ids, B, pairs, sc, 1e-4, stages=stages)
    g, meta = gpu_util.gpu_closest_hit(rays, ids, B, pairs, sc, 1e-4)
    assert np.array_equal(g[0], ref[0])
    for a, b in zip(g[1:], ref[1:]):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    leaf = pairs[1].astype(np.int64)
    assert int(meta.final_tests) == int(np.minimum(B, n - leaf * B).sum())
    assert (int(meta.final_u_pass), int(meta.final_uv_pass)) == (stages["u"], stages["uv"])
    if n_pairs > 1000:
        assert stages["u"] > 100 and (ref[0] >= 0).sum() > 10
