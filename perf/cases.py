"""Performance cases of the CRSH path: what a renderer has it do, through the
public entry points (``pipeline``, ``batch``, ``autograd`` and the C-ABI
binding), over the range of frames it is used for.

Kinds of case:

* ``frame``   one frame, hash -> sort -> build -> traverse -> closest hit
              (``pipeline.run_frame``), with the pairs stored (the default),
              the last level fused with the final tests, or packed pairs over
              triangle batches;
* ``bounce``  two generations of secondary rays: the second from the closest
              hits of the first;
* ``batch``   many uneven frames at once, enqueued or replayed as one graph;
* ``grad``    a step of a differentiable renderer: closest hits of given rays
              and the gradients of the vertices, origins and directions;
* ``sort``    the ray sort alone.

Scenes are procedural (``workloads.meshes``); the primary-hit buffers are cast
here with torch on the GPU in float64, so that new inputs are cheap.
"""
import math

import numpy as np
import torch

from paper_2312_06538_amd import crsh as X
from paper_2312_06538_amd import pipeline as P
from paper_2312_06538_amd.autograd import ClosestHit, RayScene
from paper_2312_06538_amd.batch import DeviceBatch
from workloads import meshes
from workloads.scenes import MAT_REFLECT, MAT_REFRACT, REFLECT, REFRACT, SHADOW, Scene, Workload

F64 = torch.float64
EPS = 1e-3            # ray offset off the surface, and shadow rays' end before it
T_MIN = 1e-4


def listed():
    return [
        # a small shadow pass, as for one light of a preview: every stage is a
        # launch of a few thousand items
        {"name": "shadow_128", "kind": "frame", "scene": "shadow", "w": 128, "h": 128, "meshes": 4,
         "B": 8, "F": 4, "n": 4, "path": "stored"},
        # a thumbnail of a scene with every ray type; ragged tails everywhere
        {"name": "mixed_128x72", "kind": "frame", "scene": "mixed", "w": 128, "h": 72, "meshes": 48,
         "B": 16, "F": 4, "n": 6, "path": "stored"},
        # the square megapixel frame, shadow and reflection rays
        {"name": "refl_1024", "kind": "frame", "scene": "refl", "w": 1024, "h": 1024, "meshes": 64,
         "B": 16, "F": 4, "n": 5, "path": "stored"},
        # the full-HD frame with two lights, reflection and refraction
        {"name": "mixed_1080p", "kind": "frame", "scene": "mixed", "w": 1920, "h": 1080, "meshes": 256,
         "B": 16, "F": 4, "n": 6, "path": "stored"},
        # an odd window size with wide bundles and wide nodes
        {"name": "refl_odd_wide", "kind": "frame", "scene": "refl", "w": 509, "h": 383, "meshes": 37,
         "B": 32, "F": 8, "n": 3, "path": "stored"},
        # a memory-tight render: the level-1 pairs are never stored
        {"name": "mixed_360p_fused", "kind": "frame", "scene": "mixed", "w": 640, "h": 360, "meshes": 96,
         "B": 16, "F": 4, "n": 5, "path": "fused"},
        # the paper's evaluation shape (512 x 512, depth 2, subdivision 8) with
        # its 32-bit pairs
        {"name": "refl_512_packed", "kind": "frame", "scene": "refl", "w": 512, "h": 512, "meshes": 32,
         "B": 8, "F": 8, "n": 2, "path": "packed"},
        # reflections of reflections
        {"name": "bounce_512", "kind": "bounce", "scene": "refl", "w": 512, "h": 512, "meshes": 64,
         "B": 16, "F": 4, "n": 5},
        # a serving batch of uneven frames as one graph launch
        {"name": "batch_24", "kind": "batch", "frames": 24, "max_rays": 1 << 20, "max_tris": 200000,
         "B": 16, "F": 4, "n": 5, "graph": True},
        # a small and a full step of an optimisation over vertices
        {"name": "grad_96", "kind": "grad", "w": 96, "h": 96, "spheres": 4, "sub": 2, "B": 16, "F": 4, "n": 5},
        {"name": "grad_512", "kind": "grad", "w": 512, "h": 512, "spheres": 16, "sub": 3, "B": 16, "F": 4, "n": 5},
        # a large ray sort on its own
        {"name": "sort_16m", "kind": "sort", "rays": (1 << 24) + 4097},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# hierarchy shapes (bundle, merge factor, levels) in use: the workloads', the
# paper's, and the tuner's and tests' other points
SHAPES = [(8, 4, 4), (16, 4, 5), (16, 4, 6), (8, 4, 3), (32, 8, 3), (4, 4, 6), (32, 2, 7), (16, 16, 3), (8, 8, 2)]


def draw(rng):
    kind = rng.choice(["frame"] * 6 + ["bounce", "batch", "grad", "sort"])
    if kind == "sort":
        return {"kind": kind, "rays": _log(rng, 1 << 12, 1 << 24)}
    if kind == "grad":
        s = _log(rng, 48, 512)
        return {"kind": kind, "w": s, "h": max(8, s - rng.randrange(0, s // 2)), "spheres": rng.randint(1, 16),
                "sub": rng.choice([2, 3]), "B": rng.choice([8, 16]), "F": 4, "n": rng.randint(3, 6)}
    if kind == "batch":
        B, F, n = rng.choice(SHAPES[:5])
        return {"kind": kind, "frames": rng.randint(2, 20), "max_rays": _log(rng, 1 << 14, 1 << 19),
                "max_tris": _log(rng, 2000, 100000), "B": B, "F": F, "n": n, "graph": rng.random() < 0.5}
    B, F, n = rng.choice(SHAPES)
    flat = n <= 3
    path = rng.choice(["stored"] * 3 + ["fused", "packed"])
    most = 400 if flat or path == "packed" or kind == "bounce" else 1000
    px = _log(rng, 64 * 64, most * most)
    w = max(16, int(math.sqrt(px * rng.uniform(0.6, 1.9))))
    c = {"kind": kind, "scene": "refl" if kind == "bounce" else rng.choice(["shadow", "refl", "mixed"]), "w": w,
         "h": max(16, px // w), "meshes": _log(rng, 2, 48 if flat or path == "packed" else 128), "B": B, "F": F, "n": n}
    if kind == "frame":
        c["path"] = path
    return c


# ------------------------------------------------------------------- scenes
_ICO = {}


def _ico(sub):
    if sub not in _ICO:
        _ICO[sub] = meshes.icosphere(sub)
    return _ICO[sub]


def _any_mesh(rng, torus):
    fam = int(rng.integers(0, 3))
    if fam == 0:
        return _ico(3)
    return meshes.torus(*torus) if fam == 1 else meshes.displaced_grid(32, rng)


def _placed(v, rng, center):
    return (v @ meshes.random_rotation(rng).T) * rng.lognormal(0.0, 0.5) + center


def _ball(v):
    """An enclosing sphere of float32 vertices (bounding-box centre)."""
    v = v.astype(np.float64)
    c = (0.5 * (v.min(0) + v.max(0))).astype(np.float32)
    r = np.sqrt(((v - c.astype(np.float64)) ** 2).sum(1).max()) * (1 + 2.0 ** -19) + 2.0 ** -19 * np.abs(c).max()
    return [c[0], c[1], c[2], np.nextafter(np.float32(r), np.float32(np.inf))]


def _scene(parts, mats, flags, ior):
    tris, first, count, balls, at = [], [], [], [], 0
    for v, f in parts:
        v = v.astype(np.float32)
        tris.append(v[f])
        first.append(at)
        count.append(len(f))
        at += len(f)
        balls.append(_ball(v))
    return Scene(tris=np.ascontiguousarray(np.concatenate(tris)), mesh_first=np.array(first, np.uint32),
                 mesh_count=np.array(count, np.uint32), mesh_sphere=np.array(balls, np.float32),
                 mesh_mat=np.array(mats, np.int32), mat_flags=np.array(flags, np.uint32),
                 mat_ior=np.array(ior, np.float32))


def _shadow_scene(rng, n):
    v, f = _ico(2)
    parts = [(v * rng.uniform(0.5, 1.5) + rng.uniform(-3.0, 3.0, size=3), f) for _ in range(n)]
    parts += meshes.room_walls([-50, -4, -50], [50, 40, 50], 1)     # every pixel hits
    return dict(scene=_scene(parts, [0] * len(parts), [0], [1.0]), eye=[0.37, 2, 12], lights=[[5, 10, 5]],
                ray_types=SHADOW)


def _refl_scene(rng, n, sub=8):
    parts = [(_placed(v, rng, rng.uniform(-10.0, 10.0, size=3)), f)
             for v, f in (_any_mesh(rng, (32, 16)) for _ in range(n))]
    parts += meshes.room_walls([-30, -16, -30], [30, 30, 42], sub)
    return dict(scene=_scene(parts, [0] * len(parts), [MAT_REFLECT], [1.0]), eye=[0.37, 8, 38], lights=[[15, 25, 15]],
                ray_types=SHADOW | REFLECT)


def _mixed_scene(rng, n):
    means = rng.uniform(-10.0, 10.0, size=(8, 3))
    parts, mats = [], []
    for _ in range(n):
        v, f = _any_mesh(rng, (48, 24))
        parts.append((_placed(v, rng, means[int(rng.integers(0, 8))] + rng.normal(0.0, 3.0, size=3)), f))
        mats.append(1 if rng.uniform() < 0.25 else 0)
    walls = meshes.room_walls([-35, -18, -35], [35, 32, 50], 8)
    return dict(scene=_scene(parts + walls, mats + [0] * len(walls), [MAT_REFLECT, MAT_REFRACT], [1.0, 1.5]),
                eye=[0.37, 10, 45], lights=[[15, 25, 15], [-20, 22, -10]], ray_types=SHADOW | REFLECT | REFRACT)


SCENES = {"shadow": _shadow_scene, "refl": _refl_scene, "mixed": _mixed_scene}


# ------------------------------------------------- primary hits (float64, GPU)
def _cross(a, b):
    return torch.linalg.cross(a, b, dim=-1)


def _pixel_dirs(W, H, eye, vfov=45.0):
    f = -eye / eye.norm()                      # the cameras look at the origin
    r = _cross(f, torch.tensor([0.0, 1.0, 0.0], dtype=F64, device="cuda"))
    r = r / r.norm()
    u = _cross(r, f)
    th = math.tan(math.radians(vfov) / 2.0)
    xs = ((torch.arange(W, dtype=F64, device="cuda") + 0.5) / W * 2.0 - 1.0) * (th * W / H)
    ys = (1.0 - (torch.arange(H, dtype=F64, device="cuda") + 0.5) / H * 2.0) * th
    d = f + xs[None, :, None] * r + ys[:, None, None] * u
    return (d / d.norm(dim=-1, keepdim=True)).reshape(-1, 3), (f, r, u, th)


def cast_primary(tris, W, H, eye, chunk=1 << 23):
    """Nearest triangle through every pixel centre: (triangle id or -1, hit
    point, unit normal facing the eye), float64 on the GPU."""
    tris = torch.as_tensor(tris).cuda().to(F64)
    eye = torch.tensor(eye, dtype=F64, device="cuda")
    dirs, (f, r, u, th) = _pixel_dirs(W, H, eye)
    rel = tris - eye
    x, y, z = rel @ r, rel @ u, rel @ f
    # screen box of every triangle; one that crosses the eye's plane may cover
    # any pixel
    sx = ((x / z) / (th * W / H) + 1.0) * (0.5 * W) - 0.5
    sy = (1.0 - (y / z) / th) * (0.5 * H) - 0.5
    front = z > 1e-4
    part = front.any(1) & ~front.all(1)
    lim = lambda v, n: v.clamp(-4.0, n + 4.0)
    x0 = torch.where(part, -4.0, lim(sx.amin(1).floor() - 1, W))
    x1 = torch.where(part, W + 4.0, lim(sx.amax(1).ceil() + 1, W))
    y0 = torch.where(part, -4.0, lim(sy.amin(1).floor() - 1, H))
    y1 = torch.where(part, H + 4.0, lim(sy.amax(1).ceil() + 1, H))
    seen = front.any(1) & (x1 >= 0) & (x0 <= W - 1) & (y1 >= 0) & (y0 <= H - 1)
    ids = seen.nonzero().flatten()
    bx = x0[ids].clamp(0, W - 1).long()
    by = y0[ids].clamp(0, H - 1).long()
    bw = x1[ids].clamp(0, W - 1).long() - bx + 1
    area = bw * (y1[ids].clamp(0, H - 1).long() - by + 1)
    csum = area.cumsum(0).cpu().numpy()
    e1, e2 = tris[:, 1] - tris[:, 0], tris[:, 2] - tris[:, 0]
    T = eye - tris[:, 0]
    # with the eye as origin, the numerators are dot products with the
    # direction: det = d . n, u det = d . a, v det = d . b, t det = c
    n, a, b = _cross(e2, e1), _cross(e2, T), _cross(T, e1)
    c = (e2 * b).sum(1)
    best = torch.full((W * H,), (1 << 63) - 1, dtype=torch.int64, device="cuda")
    s = 0
    while s < len(csum):
        base = int(csum[s - 1]) if s else 0
        e = max(int(np.searchsorted(csum, base + chunk, side="right")), s + 1)
        k = torch.repeat_interleave(torch.arange(s, e, device="cuda"), area[s:e])
        local = torch.arange(k.numel(), device="cuda") - (area.cumsum(0) - area)[k] + base
        pix = (by[k] + torch.div(local, bw[k], rounding_mode="floor")) * W + bx[k] + local % bw[k]
        t_id = ids[k]
        d = dirs[pix]
        det = (d * n[t_id]).sum(1)
        uu, vv, tt = (d * a[t_id]).sum(1) / det, (d * b[t_id]).sum(1) / det, c[t_id] / det
        # a little more than the triangle, so that no pixel falls between two
        ok = (det != 0) & (uu >= -1e-9) & (vv >= -1e-9) & (uu + vv <= 1 + 1e-9) & (tt > 1e-9)
        key = (tt[ok].float().view(torch.int32).long() << 32) | t_id[ok]
        best.scatter_reduce_(0, pix[ok], key, "amin")
        s = e
    hit = best != (1 << 63) - 1
    tri = torch.where(hit, best & 0xFFFFFFFF, -1)
    k = tri.clamp(min=0)
    t = c[k] / (dirs * n[k]).sum(1)
    p = torch.where(hit[:, None], eye + t[:, None] * dirs, 0.0)
    nn = n[k] / n[k].norm(dim=1, keepdim=True)
    nn = torch.where((nn * dirs).sum(1, keepdim=True) > 0, -nn, nn)
    return tri, p, torch.where(hit[:, None], nn, 0.0), dirs


def _box(tris):
    lo = (tris.reshape(-1, 3).min(0).astype(np.float64) - 1e-3).astype(np.float32)
    hi = (tris.reshape(-1, 3).max(0).astype(np.float64) + 1e-3).astype(np.float32)
    return lo, (np.float32(1.0) / (hi - lo)).astype(np.float32)


def _workload(made, W, H, seed, B, F, n):
    sc = made["scene"]
    tri, p, nn, _ = cast_primary(sc.tris, W, H, made["eye"])
    mats = torch.as_tensor(sc.tri_mat()).cuda()
    p, nn = p.float().cpu().numpy(), nn.float().cpu().numpy()
    g = {k: np.ascontiguousarray(p[:, i]) for i, k in enumerate(("px", "py", "pz"))}
    g.update({k: np.ascontiguousarray(nn[:, i]) for i, k in enumerate(("nx", "ny", "nz"))})
    g["mat"] = torch.where(tri >= 0, mats[tri.clamp(min=0)].long(), -1).to(torch.int32).cpu().numpy()
    lo, inv = _box(sc.tris)
    return Workload(name="frame", seed=seed, scene=sc, W=W, H=H, eye=np.array(made["eye"], np.float32),
                    look=np.zeros(3, np.float32), vfov=45.0, lights=np.array(made["lights"], np.float32), gbuf=g,
                    B=B, F=F, n=n, ray_types=made["ray_types"], eps_off=EPS, eps_shadow=EPS, t_min=T_MIN, lo=lo,
                    inv_ext=inv)


def _frame_workload(c, seed):
    rng = np.random.default_rng(seed)
    return _workload(SCENES[c["scene"]](rng, c["meshes"]), c["w"], c["h"], seed, c["B"], c["F"], c["n"])


def _batch_workloads(c, seed):
    """Frames of 4096 to max_rays rays and 1000 to max_tris triangles, both
    spread evenly over their logarithms, in an order that mixes them."""
    rng = np.random.default_rng(seed)
    size = np.random.default_rng(c["frames"])
    at = [(size.permutation(c["frames"]) + 0.5) / c["frames"] for _ in range(2)]
    out = []
    for k in range(c["frames"]):
        rays = 4096.0 * (c["max_rays"] / 4096.0) ** at[0][k]
        tris = 1000.0 * (c["max_tris"] / 1000.0) ** at[1][k]
        side = max(8, int(math.ceil(math.sqrt(rays / 2.0))))
        made = _refl_scene(rng, max(1, int(round(tris / 1450.0))), sub=4)
        out.append(_workload(made, side, side, seed, c["B"], c["F"], c["n"]))
    return out


def _grad_inputs(c, seed):
    """Displaced icospheres (indexed) and the reflection rays of a view of
    them, with the loss's gradients of t, u and v."""
    rng = np.random.default_rng(seed)
    vs, fs = _ico(c["sub"])
    verts, faces, first = [], [], []
    for k in range(c["spheres"]):
        noise = meshes.value_noise3(rng, freq=2.0)
        v = vs * (1.0 + 0.1 * noise(vs))[:, None]
        verts.append((v * rng.uniform(0.5, 1.5) + rng.uniform(-6.0, 6.0, size=3)).astype(np.float32))
        faces.append(fs + k * len(vs))
        first.append(k * len(fs))
    verts, faces = np.concatenate(verts), np.concatenate(faces).astype(np.int32)
    tri, p, nn, d = cast_primary(verts[faces], c["w"], c["h"], [0, 2, 18])
    # a fixed number of rays, spread evenly over the pixels that hit
    hit = (tri >= 0).nonzero().flatten()
    n = c["w"] * c["h"] // 4
    hit = hit[torch.arange(n, device="cuda") * hit.numel() // n]
    p, nn, d = p[hit], nn[hit], d[hit]
    d = d - 2.0 * (d * nn).sum(1, keepdim=True) * nn
    gen = torch.Generator(device="cuda").manual_seed(seed)
    g = [torch.randn(p.shape[0], device="cuda", generator=gen) for _ in range(3)]
    lo, inv = _box(verts[faces])
    return dict(verts=torch.as_tensor(verts).cuda(), faces=faces, first=np.array(first, np.uint32),
                count=np.full(c["spheres"], len(fs), np.uint32), lo=lo, inv=inv,
                o=(p + EPS * nn).float(), d=(d / d.norm(dim=1, keepdim=True)).float(), g=g)


def _sort_keys(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    # 30 random bits under the two type bits of the rays' keys
    k = torch.randint(0, 3 << 30, (c["rays"],), dtype=torch.int64, device="cuda", generator=gen)
    return torch.where(k >= 1 << 31, k - (1 << 32), k).to(torch.int32)


# --------------------------------------------------------------- the passes
_STREAM = []


def _side_stream():
    """The one stream that batches are captured and replayed on."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    return _STREAM[0]


def prepare(case, seed):
    c = dict(case)
    st = {"case": c}
    if c["kind"] in ("frame", "bounce"):
        fr = P.DeviceFrame(_frame_workload(c, seed))
        st["fr"] = fr
        hint = max(1 << 16, 64 * fr.max_rays)
        if c["kind"] == "frame":
            bf = P.Buffers(fr, hint)
            st["bf"], m = P.run_with_retry(fr, bf, leaf_hit=c["path"] == "fused", packed=c["path"] == "packed")
            st["n"] = int(m.n_rays)
        else:
            gens = P.run_generations(fr, 2, pair_capacity=hint)
            st["bfs"] = [b for b, _ in gens]
            # a reflection ray spawns two rays, or none if it slips through a
            # seam: the places after the last ray are zeros
            st["n"] = 2 * c["w"] * c["h"]
            for b, m in gens:
                for a in (b.hit_tri, b.hit_t, b.hit_u, b.hit_v, b.sids, b.keys):
                    a[int(m.n_rays):].zero_()
    elif c["kind"] == "batch":
        b = DeviceBatch(_batch_workloads(c, seed), c["B"], c["F"], c["n"])
        m = b.run_with_retry()
        st["b"], st["n"] = b, int(m.n_rays)
        if c["graph"]:
            torch.cuda.synchronize()
            st["graph"] = b.graph(_side_stream())
    elif c["kind"] == "grad":
        i = _grad_inputs(c, seed)
        st["scene"] = RayScene(i["faces"], i["first"], i["count"], i["lo"], i["inv"], B=c["B"], F=c["F"],
                               levels=c["n"], t_min=T_MIN, ray_type=1)
        st["in"] = [i[k].requires_grad_(True) for k in ("verts", "o", "d")]
        st["g"] = i["g"]
    else:
        keys = _sort_keys(c, seed)
        n = c["rays"]
        e = lambda: torch.empty(n, dtype=torch.int32, device="cuda")
        meta = X.Meta()
        meta.n_rays = n
        st["meta"] = torch.from_numpy(np.frombuffer(bytes(meta), np.uint8).copy()).cuda()
        st["wsb"] = X.crsh_workspace_size(n, 1, 1, 1, 1)
        st["ws"] = torch.empty(st["wsb"], dtype=torch.uint8, device="cuda")
        st["keys"] = (keys, torch.arange(n, dtype=torch.int32, device="cuda"), e(), e())
    return st


def _hits(b, n):
    return {"tri": b.hit_tri[:n], "t": b.hit_t[:n], "u": b.hit_u[:n], "v": b.hit_v[:n], "order": b.sids[:n],
            "keys": b.keys[:n]}


def run(st):
    c = st["case"]
    if c["kind"] == "frame":
        P.run_frame(st["fr"], st["bf"], leaf_hit=c["path"] == "fused", packed=c["path"] == "packed")
        return _hits(st["bf"], st["n"])
    if c["kind"] == "bounce":
        b0, b1 = st["bfs"]
        P.run_frame(st["fr"], b0)
        P.run_frame(st["fr"], b1, parent=b0)
        return [_hits(b0, st["n"]), _hits(b1, st["n"])]
    if c["kind"] == "batch":
        if c["graph"]:
            st["graph"].launch()
        else:
            st["b"].enqueue()
        return _hits(st["b"], st["n"])
    if c["kind"] == "grad":
        tri, t, u, v = ClosestHit.apply(*st["in"], st["scene"])
        gv, go, gd = torch.autograd.grad([t, u, v], st["in"], st["g"])
        return {"tri": tri, "t": t, "u": u, "v": v, "g_verts": gv, "g_o": go, "g_d": gd}
    k, i, ko, io = st["keys"]
    X.crsh_sort(k.data_ptr(), i.data_ptr(), ko.data_ptr(), io.data_ptr(), c["rays"], st["meta"].data_ptr(),
                st["ws"].data_ptr(), st["wsb"], P.stream_handle())
    return {"keys": ko, "ids": io}


# ----------------------------------------------------------------- the floor
def _tris(c):
    """About the triangles of the case's scene."""
    if c["kind"] == "grad":
        return c["spheres"] * 20 * 4 ** c["sub"]
    per, room = {"shadow": (320, 12), "refl": (1450, 768), "mixed": (1877, 768)}[c["scene"]]
    return per * c["meshes"] + room


def work(case):
    """Bytes: primary hits (28 B a pixel) or rays (24 B) and triangles (36 B)
    read once, hits, order and keys (24 B a ray) written once.  Operations:
    one ray-triangle test (53) and one ray made and hashed (about 80) a ray;
    how many further tests a frame needs depends on the scene."""
    c = case
    if c["kind"] == "sort":
        return {"bytes": 16 * c["rays"], "flops": 0}
    if c["kind"] == "grad":
        n = c["w"] * c["h"] // 4
        return {"bytes": n * (24 + 16 + 12 + 24) + _tris(c) * (12 + 6 + 6), "flops": n * (53 + 90)}
    if c["kind"] == "batch":
        lm = lambda lo, hi: (hi - lo) / math.log(hi / lo)     # the mean of a log-uniform size
        rays = c["frames"] * lm(4096.0, c["max_rays"] + 1.0)
        return {"bytes": rays * 14 + c["frames"] * lm(1000.0, c["max_tris"] + 1.0) * 36 + rays * 24,
                "flops": rays * 133}
    px = c["w"] * c["h"]
    rays = px * {"shadow": 1, "refl": 2, "mixed": 3}[c["scene"]]
    gens = 2 if c["kind"] == "bounce" else 1
    return {"bytes": px * 28 + _tris(c) * 36 + gens * rays * 24, "flops": gens * rays * 133}


# ------------------------------------------------------- exact values (64 bit)
def _closest64(o, d, tmax, tris, chunk=1 << 26):
    """t, u, v and the triangle (-1: none) of the nearest two-sided hit with
    T_MIN < t < tmax, all pairs in float64."""
    v0 = tris[:, 0]
    e1, e2 = tris[:, 1] - v0, tris[:, 2] - v0
    n = _cross(e2, e1)                          # det = d . n
    mom = torch.cat([_cross(o, d), d], 1)
    wu = torch.cat([e2, -_cross(e2, v0)], 1).T.contiguous()
    wv = torch.cat([-e1, -_cross(v0, e1)], 1).T.contiguous()
    nt, c0 = n.T.contiguous(), (v0 * n).sum(1)
    best_t = torch.full((o.shape[0],), math.inf, dtype=F64, device="cuda")
    best = torch.full((o.shape[0],), -1, dtype=torch.int64, device="cuda")
    step = max(1, min(o.shape[0], chunk // max(1, min(len(tris), 4096))))
    for r in range(0, o.shape[0], step):
        s = slice(r, r + step)
        for k in range(0, len(tris), 4096):
            q = slice(k, k + 4096)
            inv = 1.0 / (d[s] @ nt[:, q])
            u, v, t = (mom[s] @ wu[:, q]) * inv, (mom[s] @ wv[:, q]) * inv, (c0[q] - o[s] @ nt[:, q]) * inv
            ok = (u >= 0) & (v >= 0) & (u + v <= 1) & (t > T_MIN) & (t < tmax[s, None])
            t, at = torch.where(ok, t, math.inf).min(1)
            near = t < best_t[s]
            best_t[s] = torch.where(near, t, best_t[s])
            best[s] = torch.where(near, at + k, best[s])
    hit = best >= 0
    k = best.clamp(min=0)
    det = (d * n[k]).sum(1)
    u, v = ((mom * w.T[k]).sum(1) / det for w in (wu, wv))
    z = lambda x: torch.where(hit, x, 0.0)
    return best, z(best_t), z(u), z(v)


def _rays64(wl):
    """The secondary rays of a frame in (pixel, slot) order, float64."""
    g = {k: torch.as_tensor(v).cuda() for k, v in wl.gbuf.items()}
    p = torch.stack([g["px"], g["py"], g["pz"]], 1).to(F64)
    nn = torch.stack([g["nx"], g["ny"], g["nz"]], 1).to(F64)
    mat = g["mat"].long()
    flags = torch.as_tensor(wl.scene.mat_flags.astype(np.int64)).cuda()[mat.clamp(min=0)]
    ior = torch.as_tensor(wl.scene.mat_ior).cuda().to(F64)[mat.clamp(min=0)]
    hit = mat >= 0
    big = torch.full((len(mat),), float(np.finfo(np.float32).max), dtype=F64, device="cuda")
    slots = []
    for L in torch.as_tensor(wl.lights).cuda().to(F64):
        s = p - L
        r = s.norm(dim=1)
        slots.append((L.expand_as(p), s / r[:, None], r - EPS, hit & bool(wl.ray_types & SHADOW)))
    v = p - torch.as_tensor(wl.eye).cuda().to(F64)
    v = v / v.norm(dim=1, keepdim=True)
    cos = (v * nn).sum(1, keepdim=True)
    slots.append((p + EPS * nn, v - 2.0 * cos * nn, big,
                  hit & ((flags & MAT_REFLECT) != 0) & bool(wl.ray_types & REFLECT)))
    eta = (1.0 / ior)[:, None]
    k = 1.0 - eta * eta * (1.0 - cos * cos)
    slots.append((p - EPS * nn, eta * v - (eta * cos + k.clamp(min=0).sqrt()) * nn, big,
                  hit & ((flags & MAT_REFRACT) != 0) & (k[:, 0] >= 0) & bool(wl.ray_types & REFRACT)))
    keep = torch.stack([s[3] for s in slots], 1).flatten()
    pick = lambda i: torch.stack([s[i] for s in slots], 1).flatten(0, 1)[keep]
    return pick(0), pick(1), pick(2)


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "frame":
        rays = c["w"] * c["h"] * {"shadow": 1, "refl": 2, "mixed": 3}[c["scene"]]
        if rays * _tris(c) > 4e10:
            return None
        wl = _frame_workload(c, seed)
        o, d, tmax = _rays64(wl)
        _, t, u, v = _closest64(o, d, tmax, torch.as_tensor(wl.scene.tris).cuda().to(F64))
        return {"tri": None, "t": t, "u": u, "v": v, "order": None, "keys": None}
    if c["kind"] == "grad":
        i = _grad_inputs(c, seed)
        verts, faces = i["verts"].to(F64), torch.as_tensor(i["faces"]).cuda().long()
        o, d = i["o"].to(F64), i["d"].to(F64)
        tris = verts[faces]
        tmax = torch.full((o.shape[0],), float(np.finfo(np.float32).max), dtype=F64, device="cuda")
        tri, t, u, v = _closest64(o, d, tmax, tris)
        hit = (tri >= 0)[:, None]
        k = tri.clamp(min=0)
        e1, e2 = tris[k, 1] - tris[k, 0], tris[k, 2] - tris[k, 0]
        # o + t d = (1-u-v) v0 + u v1 + v v2, differentiated with the triangle
        # held fixed: the adjoint solves the transposed 3 x 3 system
        A = torch.stack([d, -e1, -e2], 1)      # rows: the transposed columns
        A = torch.where(hit[..., None], A, torch.eye(3, dtype=F64, device="cuda"))
        g = torch.stack([x.to(F64) for x in i["g"]], 1)
        lam = torch.where(hit, torch.linalg.solve(A, g[..., None])[..., 0], 0.0)
        gv = torch.zeros_like(verts)
        for j, w in enumerate((1.0 - u - v, u, v)):
            gv.index_add_(0, faces[k, j], w[:, None] * lam)
        return {"tri": None, "t": t, "u": u, "v": v, "g_verts": gv, "g_o": -lam, "g_d": -t[:, None] * lam}
    return None
