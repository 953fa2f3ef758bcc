"""The final tests' matrix filter where lengths are far from 1: directions of
any length, and edges and distances up to and past the ends of its range -- every
hit and counter exactly the oracle's; and that such rays are still rejected by
it, shown by the time their tests take."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _case(seed, n, m, n_pairs, B, place, size, length, at=0.0):
    """Triangles of about `size` within `place` of the point (at, at, at), rays
    aimed at, on and beside their edges, directions of about `length`; each of
    the three a number, or a range of exponents of two that is drawn from."""
    from workloads.scenes import Scene
    rng = np.random.default_rng(seed)
    of = lambda x, k: np.exp2(rng.uniform(*x, (k, 1))) if isinstance(x, tuple) else np.full((k, 1), float(x))
    e, far = of(size, m), of(place, m)
    v0 = rng.uniform(-1, 1, (m, 3)) * far + at
    tris = np.stack([v0, v0 + rng.normal(0, 1, (m, 3)) * e, v0 + rng.normal(0, 1, (m, 3)) * e], 1).astype(np.float32)
    o = (rng.uniform(-1, 1, (n, 3)) * of(place, n) + at).astype(np.float32)
    k = rng.integers(0, m, n)
    t = tris[k].astype(np.float64)
    u = np.where(rng.random(n) < 0.5, 0.0, 1.0) + rng.normal(size=n) * np.exp2(rng.uniform(-26, 1, n))
    p = t[:, 0] + u[:, None] * (t[:, 1] - t[:, 0]) + rng.uniform(0, 1, (n, 1)) * (t[:, 2] - t[:, 0])
    d = p - o
    d = (d / np.maximum(np.linalg.norm(d, axis=1, keepdims=True), 1e-300) * of(length, n)).astype(np.float32)
    sc = Scene(tris=tris, mesh_first=np.zeros(1, np.uint32), mesh_count=np.array([m], np.uint32),
               mesh_sphere=np.array([[0, 0, 0, 1e30]], np.float32), mesh_mat=np.zeros(1, np.int32),
               mat_flags=np.zeros(1, np.uint32), mat_ior=np.ones(1, np.float32))
    rays = {"ox": o[:, 0], "oy": o[:, 1], "oz": o[:, 2], "dx": d[:, 0], "dy": d[:, 1], "dz": d[:, 2],
            "tmax": np.full(n, np.finfo(np.float32).max, np.float32), "pix": np.zeros(n, np.uint32)}
    leaves = -(-n // B)
    # half of a leaf's pairs with the triangles its rays are aimed at
    node = rng.integers(0, leaves, n_pairs)
    tri = np.where(rng.random(n_pairs) < 0.5, k[np.minimum(node * B + rng.integers(0, B, n_pairs), n - 1)],
                   rng.integers(0, m, n_pairs))
    return sc, rays, (tri.astype(np.uint32), node.astype(np.uint32))


# place, edge length, direction length: at, inside and past 2^40 and 2^-40
@pytest.mark.parametrize("B,place,size,length", [
    (4, 20.0, 1.0, (-46, 46)), (16, 20.0, 1.0, (-12, -8)), (8, 20.0, 1.0, (-42, -38)), (16, 20.0, 1.0, (38, 42)),
    (32, 20.0, (-44, 10), 1.0), (16, (15, 44), (15, 44), (-40, -30)), (5, (30, 42), (38, 41), (20, 41)),
    (16, (-44, 0), (-44, 0), (-40, 40)), (1, (-45, 45), (-45, 45), (-45, 45)), (17, 1e-3, 1e-4, (-30, 0))])
def test_lengths_match_oracle(B, place, size, length):
    import gpu_util
    n, m, n_pairs = 6000, 400, 60000
    sc, rays, pairs = _case(B, n, m, n_pairs, B, place, size, length)
    ids = np.random.default_rng(B).permutation(n).astype(np.uint32)
    inv = np.empty(n, np.int64)
    inv[ids] = np.arange(n)
    rays = {k: v[inv] for k, v in rays.items()}          # ray ids[s] is sorted ray s
    stages = {}
    ref = O.closest_hit(rays, ids, B, pairs, sc, 1e-4, stages=stages)
    g, meta = gpu_util.gpu_closest_hit(rays, ids, B, pairs, sc, 1e-4)
    print(f"[hit lengths] B={B} {place} {size} {length}: u {stages['u']} hits {(ref[0] >= 0).sum()}", flush=True)
    for a, b in zip(g, ref):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    assert (int(meta.final_u_pass), int(meta.final_uv_pass)) == (stages["u"], stages["uv"])


def _hit_us(place, size, length, at=0.0, n=1 << 16, m=2000, n_pairs=1 << 23, B=16):
    """Final tests with no hits, all of the triangles drawn alike."""
    import gpu_util
    import torch
    from paper_2312_06538_amd import crsh as X
    sc, rays, _ = _case(2, n, m, 16, B, place, size, length, at)
    rays["tmax"][:] = 0.0
    gen = torch.Generator(device="cuda").manual_seed(5)
    # pairs in runs of 256 neighbouring leaves, as a hierarchy gives them
    node = (torch.arange(n_pairs, device="cuda") >> 13) % (n // B // 256) * 256
    node = (node + torch.randint(0, 256, (n_pairs,), device="cuda", generator=gen)).to(torch.int32)
    tri = torch.randint(0, m, (n_pairs,), device="cuda", generator=gen, dtype=torch.int32)
    r = {k: gpu_util.dev_f32(rays[k]) for k in gpu_util.RAY_KEYS}
    c_r = X.Rays(*[r[k].data_ptr() for k in gpu_util.RAY_KEYS], None, n)
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    pairs = X.Pairs(tri.data_ptr(), node.data_ptr(), n_pairs)
    c_sc, keep = gpu_util._scene(sc)
    out = [torch.zeros(n, dtype=dt, device="cuda") for dt in (torch.int64, torch.int32, *[torch.float32] * 3)]
    hits = X.Hits(*[x.data_ptr() for x in out], n)
    meta = gpu_util.new_meta(n_rays=n, n_levels=1, pairs=[n_pairs])
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


def test_short_and_long_directions_cost():
    """The same rays with directions of other lengths take the same tests: all
    in full where the filter did not take them, 6 times as long."""
    unit, short, long = _hit_us(20.0, 1.0, 1.0), _hit_us(20.0, 1.0, 2.0 ** -20), _hit_us(20.0, 1.0, 2.0 ** 30)
    print(f"[hit lengths] {unit:.0f} us, 2^-20 {short:.0f}, 2^30 {long:.0f}", flush=True)
    assert short < 1.5 * unit and long < 1.5 * unit


def test_far_scene_cost():
    """A scene takes no longer 2^20 from the origin than around it, where the
    filter's bound grew with the distance to more than the scene's size."""
    near, far = _hit_us(20.0, 2.0, 1.0), _hit_us(20.0, 2.0, 1.0, at=2.0 ** 20)
    print(f"[hit lengths] at the origin {near:.0f} us, 2^20 from it {far:.0f}", flush=True)
    assert far < 1.5 * near


@pytest.mark.parametrize("at,m,odd", [(3e4, 400, 0), (-1e6, 400, 0), (2.0 ** 39, 400, 0), (5e3, 1, 0), (5e3, 2, 0),
                                      (5e3, 3, 0), (7e3, 5, 1), (7e3, 400, 1), (7e3, 400, 2), (0.0, 400, 3)])
def test_far_scenes_match_oracle(at, m, odd):
    """Scenes far from the origin, of few triangles, and with triangles far from
    the others, infinite or no numbers where the filter takes its centre from."""
    import gpu_util
    B, n, n_pairs = 8, 3000, 30000
    sc, rays, pairs = _case(m + odd, n, m, n_pairs, B, max(20.0, abs(at) / 4096), max(0.2, abs(at) / 65536), 1.0, at)
    for k, t in enumerate((m // 4, m // 2, m - 1 - m // 4)):
        if odd == 1 and k != 1 or odd == 3:
            sc.tris[t] *= np.float32([1e7, 1e30, -1e7][k])
        if odd == 2:
            sc.tris[t, 0, k] = [np.nan, np.inf, -np.inf][k]
    stages = {}
    ids = np.arange(n, dtype=np.uint32)
    with np.errstate(all="ignore"):
        ref = O.closest_hit(rays, ids, B, pairs, sc, 1e-4, stages=stages)
    g, meta = gpu_util.gpu_closest_hit(rays, ids, B, pairs, sc, 1e-4)
    print(f"[hit lengths] at {at} m={m} odd={odd}: u {stages['u']} hits {(ref[0] >= 0).sum()}", flush=True)
    for a, b in zip(g, ref):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    assert (int(meta.final_u_pass), int(meta.final_uv_pass)) == (stages["u"], stages["uv"])
