// Stage 3: hierarchy creation (Sec. 3.3.6, Eq. 1-8).
//
// k_build_leaf  rays gathered into sorted order (coalesced writes; the final
//               tests read them so) and, from the copy of them in LDS, the
//               level-1 nodes: the compact cone of a node's B rays added one
//               at a time in sorted order (Eq. 1-4) and the sphere of their
//               origins as a balanced pairwise tree (Eq. 7-8); one thread
//               takes the node counts of every level from the ray count
//               (device side, so the frame needs no host round trip);
// k_build_up    one thread per upper node: balanced pairwise trees of its F
//               children's spheres (Eq. 7-8) and cones (Eq. 5-6);
// k_build_tail  the levels of at most UP_TAIL nodes, one block for all of them.
// Trees are unrolled over a power-of-two slot count, so every slot index is a
// compile-time constant and the nodes stay in registers.
//
// Batched form: k_batch_levels sizes every frame's levels (the same rule as
// the plain one, per frame) and lays each level out frame by frame; the leaf
// and upper kernels find their frame and take their rays / children from the
// frame's ranges, and record each node's first ray or child and its count
// (with the frame) for the traversal and the final tests.
#include "batch.hpp"
#include "bounds.hpp"

namespace crsh {

struct nodes_dev {
    float *cx, *cy, *cz, *r, *ax, *ay, *az, *c, *s, *tan, *sec;
    uint32_t cap;
};

__device__ __forceinline__ void put_sphere(const nodes_dev &nd, uint32_t i, const sph &sp)
{
    nd.cx[i] = sp.c.x;
    nd.cy[i] = sp.c.y;
    nd.cz[i] = sp.c.z;
    nd.r[i] = sp.r;
}

__device__ __forceinline__ void put_cone(const nodes_dev &nd, uint32_t i, const cone &k)
{
    nd.ax[i] = k.x.x;
    nd.ay[i] = k.x.y;
    nd.az[i] = k.x.z;
    nd.c[i] = k.c;
    nd.s[i] = k.s;
    bool open = k.c > 0.0f;
    nd.tan[i] = open ? k.s / k.c : 0.0f;
    nd.sec[i] = open ? 1.0f / k.c : 0.0f;
}

// Node counts of every level for n rays into meta (PUT); the total.
template <bool PUT>
__device__ __forceinline__ uint32_t build_info(crsh_meta *meta, uint32_t n, uint32_t B, uint32_t F, uint32_t levels,
                                               uint32_t node_cap)
{
    if (PUT) meta->n_rays = n;
    uint32_t nl = 0, total = 0;
    if (n > 0) {
        uint32_t c = (n + B - 1) / B;
        for (;;) {
            if (PUT) {
                meta->level_cnt[nl] = c;
                meta->level_off[nl] = total;
            }
            total += c;
            ++nl;
            if (nl >= levels || c <= 1) break;
            c = (c + F - 1) / F;
        }
    }
    if (PUT) {
        for (uint32_t k = nl; k < CRSH_MAX_LEVELS; ++k) {
            meta->level_cnt[k] = 0;
            meta->level_off[k] = total;
        }
        meta->nodes_required = total;
        if (total > node_cap) {
            atomicOr(&meta->status, CRSH_OVERFLOW_NODES);
            nl = 0;                      // nothing is built; the host regrows
        }
        meta->n_levels = nl;
    }
    return total;
}

// One thread per frame (at most CRSH_MAX_FRAMES frames, one block).
__global__ __launch_bounds__(256) void k_batch_levels(batch_dev bd, crsh_meta *meta, uint32_t B, uint32_t F,
                                                      uint32_t levels, uint32_t node_cap, uint32_t ray_cap)
{
    __shared__ uint32_t scratch[256 / WAVE];
    __shared__ uint32_t s_total[CRSH_MAX_LEVELS];
    __shared__ uint32_t s_nl;
    const uint32_t f = threadIdx.x;
    const bool live = f < bd.n_frames;
    const uint32_t n = min(meta->n_rays, ray_cap);
    if (f == 0) s_nl = 0;
    uint32_t rb = live ? min(bd.fm[f].ray_begin, n) : n;
    uint32_t re = (f + 1 < bd.n_frames) ? min(bd.fm[f + 1].ray_begin, n) : n;
    const uint32_t nr = (live && re > rb) ? re - rb : 0u;
    __syncthreads();
    uint32_t nl = 0, c = 0;
    for (uint32_t k = 0; k < CRSH_MAX_LEVELS; ++k) {
        // the plain rule per frame: ceil(n / B) leaves, then ceil(c / F) while
        // under `levels` levels and more than one node
        if (k == 0) {
            c = (nr + B - 1) / B;
            nl = nr ? 1u : 0u;
        } else if (nl == k && k < levels && c > 1) {
            c = (c + F - 1) / F;
            nl = k + 1;
        }
        const uint32_t ck = k < nl ? c : 0u;
        uint32_t total;
        const uint32_t base = block_excl_scan<uint32_t, 256 / WAVE>(ck, scratch, total);
        if (live) {
            bd.fm[f].level_base[k] = base;
            bd.fm[f].level_cnt[k] = ck;
        }
        if (f == 0) s_total[k] = total;
    }
    if (live) atomicMax(&s_nl, nl);
    __syncthreads();
    uint32_t total = 0;
    for (uint32_t k = 0; k < CRSH_MAX_LEVELS; ++k) total += s_total[k];
    const bool over = total > node_cap;
    if (live) {
        bd.fm[f].ray_begin = rb;
        bd.fm[f].n_rays = nr;
        bd.fm[f].n_levels = over ? 0u : nl;
    }
    if (f == 0) {
        uint32_t off = 0;
        for (uint32_t k = 0; k < CRSH_MAX_LEVELS; ++k) {
            meta->level_off[k] = off;
            meta->level_cnt[k] = s_total[k];
            off += s_total[k];
        }
        meta->n_rays = n;
        meta->nodes_required = total;
        if (over) atomicOr(&meta->status, CRSH_OVERFLOW_NODES);
        meta->n_levels = over ? 0u : s_nl;
    }
}

struct rays_in {
    const float *ox, *oy, *oz, *dx, *dy, *dz, *tmax;
    const uint32_t *pix;
};
struct rays_out {
    float *ox, *oy, *oz, *dx, *dy, *dz, *tmax;
    uint32_t *pix;
};

// A workgroup takes the rays of NODES consecutive nodes, LEAF_RAYS in all: a
// thread per ray gathers it, to memory and to LDS; then a thread per node makes
// its cone, and another its sphere, on different waves.  Gathering is bound by
// memory, the cone by a serial chain (a square root and divisions per ray):
// with workgroups of both on a compute unit one hides the other.  The ray count
// that the one writing thread stores is what every thread takes.
// (A node's places in LDS are an odd number apart: no bank conflicts.)
// Measured, against a launch that permuted the rays and one with a thread per
// node that read them back, lanes 64 bytes apart: 6.2 M rays, 16 to a node, 507
// to 235 us (2.5 TB/s of gathered reads and writes); 2.1 M 165 to 73; 24 frames
// batched 346 to 140; 16,384 rays 16 to 13, a node's chain of 8 cones.
constexpr uint32_t LEAF_THREADS = 256;
constexpr uint32_t LEAF_RAYS = 1024;
template <int NB, bool BATCH>
__global__ __launch_bounds__(LEAF_THREADS) void k_build_leaf(rays_in in, const uint32_t *__restrict__ sorted_ids,
                                                             rays_out out, uint32_t B, uint32_t F, uint32_t levels,
                                                             nodes_dev nd, crsh_meta *meta, uint32_t cap,
                                                             batch_dev bd)
{
    constexpr uint32_t NODES = LEAF_RAYS / NB;
    constexpr uint32_t ROW = NB | 1;
    __shared__ float s_ray[6][NODES * ROW];
    __shared__ uint32_t s_first[BATCH ? NODES : 1], s_cnt[BATCH ? NODES : 1];
    const uint32_t n = min(meta->n_rays, cap);
    const uint32_t j0 = blockIdx.x * NODES;
    uint32_t nodes;                         // level-1 nodes
    bool fits;                              // the hierarchy has storage
    if constexpr (BATCH) {
        nodes = meta->level_cnt[0];
        fits = meta->n_levels != 0;
    } else {
        nodes = (n + B - 1) / B;
        fits = build_info<false>(meta, n, B, F, levels, nd.cap) <= nd.cap;
        if (blockIdx.x == 0 && threadIdx.x == 0) build_info<true>(meta, n, B, F, levels, nd.cap);
    }
    if (j0 >= nodes) return;
    if constexpr (BATCH) {
        for (uint32_t q = threadIdx.x; q < NODES; q += LEAF_THREADS) {
            const uint32_t j = j0 + q;
            uint32_t b = 0u, k = 0u;
            if (j < nodes) {
                const uint32_t f = frame_of_node(bd, 0, j);
                const uint32_t local = (j - bd.fm[f].level_base[0]) * B;
                b = bd.fm[f].ray_begin + local;
                k = min(B, bd.fm[f].n_rays - local);
                if (fits) {
                    bd.node_first[j] = b;
                    bd.node_info[j] = k | (f << INFO_FRAME_SHIFT);
                }
            }
            s_first[q] = b;
            s_cnt[q] = k;
        }
        __syncthreads();
    }
    // rays of node j0 + q: sorted rays `first` on
    auto rays_of = [&](uint32_t q, uint32_t &first) {
        if constexpr (BATCH) {
            first = s_first[q];
            return s_cnt[q];
        } else {
            first = (j0 + q) * B;
            return j0 + q < nodes ? min(B, n - first) : 0u;
        }
    };
#pragma unroll
    for (uint32_t r = 0; r < LEAF_RAYS / LEAF_THREADS; ++r) {
        const uint32_t x = r * LEAF_THREADS + threadIdx.x, q = x / NB, i = x % NB;
        uint32_t first;
        if (i >= rays_of(q, first)) continue;
        const uint32_t sr = first + i;
        uint32_t id = sorted_ids[sr];
        if (id >= cap) id = 0;      // ids come from the sort: never taken
        const float v[6] = {in.ox[id], in.oy[id], in.oz[id], in.dx[id], in.dy[id], in.dz[id]};
        out.ox[sr] = v[0];
        out.oy[sr] = v[1];
        out.oz[sr] = v[2];
        out.dx[sr] = v[3];
        out.dy[sr] = v[4];
        out.dz[sr] = v[5];
        out.tmax[sr] = in.tmax[id];
        if (out.pix) out.pix[sr] = in.pix ? in.pix[id] : 0u;
#pragma unroll
        for (uint32_t k = 0; k < 6; ++k) s_ray[k][q * ROW + i] = v[k];
    }
    if (!fits) return;
    __syncthreads();
    constexpr uint32_t HALF = NODES < WAVE ? WAVE : NODES;     // cones on the first waves, spheres on the others
    for (uint32_t x = threadIdx.x; x < 2 * HALF; x += LEAF_THREADS) {
        const uint32_t q = x % HALF, at = q * ROW;
        uint32_t first;
        const uint32_t k = q < NODES ? rays_of(q, first) : 0u;
        if (k == 0u) continue;
        if (x < HALF) {
            cone kc;
            kc.x = mk(s_ray[3][at], s_ray[4][at], s_ray[5][at]);
            kc.c = 1.0f;
            kc.s = 0.0f;
            for (uint32_t i = 1; i < k; ++i)
                kc = cone_take(kc, mk(s_ray[3][at + i], s_ray[4][at + i], s_ray[5][at + i]));
            put_cone(nd, j0 + q, kc);
        } else {
            sph sp[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                if ((uint32_t)i < k) {
                    sp[i].c = mk(s_ray[0][at + i], s_ray[1][at + i], s_ray[2][at + i]);
                    sp[i].r = 0.0f;
                }
            }
#pragma unroll
            for (int w = 1; w < NB; w *= 2) {
#pragma unroll
                for (int i = 0; i + w < NB; i += 2 * w)
                    if ((uint32_t)(i + w) < k) sp[i] = merge_spheres(sp[i], sp[i + w]);
            }
            put_sphere(nd, j0 + q, sp[0]);
        }
    }
}

template <int NF, bool BATCH>
__device__ __forceinline__ void build_up(uint32_t lv, uint32_t j, uint32_t F, const nodes_dev &nd,
                                         const crsh_meta *meta, const batch_dev &bd)
{
    const uint32_t below = meta->level_off[lv - 1];
    uint32_t b, k;
    if constexpr (BATCH) {
        const uint32_t f = frame_of_node(bd, lv, j);
        const uint32_t local = (j - bd.fm[f].level_base[lv]) * F;
        b = bd.fm[f].level_base[lv - 1] + local;
        k = min(F, bd.fm[f].level_cnt[lv - 1] - local);
        bd.node_first[meta->level_off[lv] + j] = b;
        bd.node_info[meta->level_off[lv] + j] = k | (f << INFO_FRAME_SHIFT);
    } else {
        b = j * F;
        k = min(F, meta->level_cnt[lv - 1] - b);
    }
    sph sp[NF];
    cone kc[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        if ((uint32_t)i < k) {
            uint32_t q = below + b + i;
            sp[i].c = mk(nd.cx[q], nd.cy[q], nd.cz[q]);
            sp[i].r = nd.r[q];
            kc[i].x = mk(nd.ax[q], nd.ay[q], nd.az[q]);
            kc[i].c = nd.c[q];
            kc[i].s = nd.s[q];
        }
    }
#pragma unroll
    for (int w = 1; w < NF; w *= 2) {
#pragma unroll
        for (int i = 0; i + w < NF; i += 2 * w) {
            if ((uint32_t)(i + w) < k) {
                sp[i] = merge_spheres(sp[i], sp[i + w]);
                kc[i] = merge_cones(kc[i], kc[i + w]);
            }
        }
    }
    put_sphere(nd, meta->level_off[lv] + j, sp[0]);
    put_cone(nd, meta->level_off[lv] + j, kc[0]);
}

template <int NF, bool BATCH>
__global__ __launch_bounds__(256) void k_build_up(uint32_t lv, uint32_t F, nodes_dev nd, const crsh_meta *meta,
                                                  batch_dev bd)
{
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (lv >= meta->n_levels || j >= meta->level_cnt[lv]) return;
    build_up<NF, BATCH>(lv, j, F, nd, meta, bd);
}

// Levels lv0 and up, each of at most UP_TAIL nodes: a thread per node, a
// barrier between levels.  A node's chain of square roots and divisions takes
// 2 to 4 us and a launch as long again, so the upper levels of a small frame
// are one launch instead of one each.
constexpr uint32_t UP_TAIL = 512;
template <int NF, bool BATCH>
__global__ __launch_bounds__(UP_TAIL) void k_build_tail(uint32_t lv0, uint32_t F, nodes_dev nd, const crsh_meta *meta,
                                                        batch_dev bd)
{
    const uint32_t nl = meta->n_levels;
    for (uint32_t lv = lv0; lv < nl; ++lv) {
        if (threadIdx.x < meta->level_cnt[lv]) build_up<NF, BATCH>(lv, threadIdx.x, F, nd, meta, bd);
        __syncthreads();
    }
}

static int pow2_at_least(int x)
{
    int p = 1;
    while (p < x) p *= 2;
    return p;
}

}  // namespace crsh

using namespace crsh;

namespace crsh {

crsh_status build_launch(const crsh_rays *rays, const uint32_t *sorted_ids, int32_t bundle, int32_t merge,
                         int32_t levels, crsh_nodes *nodes, crsh_rays *sorted, crsh_meta *meta,
                         const batch_dev *bd, hipStream_t stream)
{
    if (!rays || !sorted_ids || !nodes || !sorted || !meta) {
        set_error("crsh_build: NULL argument");
        return CRSH_ERR_INVALID;
    }
    if (bundle < 1 || bundle > 32 || merge < 2 || merge > CRSH_MAX_MERGE || levels < 1 ||
        levels > CRSH_MAX_LEVELS) {
        set_error("crsh_build: bundle must be in [1,32], merge in [2,%d], levels in [1,%d]", CRSH_MAX_MERGE,
                  CRSH_MAX_LEVELS);
        return CRSH_ERR_INVALID;
    }
    if (!rays->ox || !rays->oy || !rays->oz || !rays->dx || !rays->dy || !rays->dz || !rays->tmax ||
        !sorted->ox || !sorted->oy || !sorted->oz || !sorted->dx || !sorted->dy || !sorted->dz || !sorted->tmax) {
        set_error("crsh_build: incomplete ray arrays");
        return CRSH_ERR_INVALID;
    }
    if (sorted->capacity < rays->capacity) {
        set_error("crsh_build: sorted-ray capacity below the ray capacity");
        return CRSH_ERR_INVALID;
    }
    if (!nodes->cx || !nodes->cy || !nodes->cz || !nodes->r || !nodes->ax || !nodes->ay || !nodes->az ||
        !nodes->c || !nodes->s || !nodes->tan || !nodes->sec) {
        set_error("crsh_build: incomplete node arrays");
        return CRSH_ERR_INVALID;
    }
    const batch_dev b = bd ? *bd : batch_dev{};
    if (bd)
        k_batch_levels<<<1, 256, 0, stream>>>(b, meta, (uint32_t)bundle, (uint32_t)merge, (uint32_t)levels,
                                               nodes->capacity, rays->capacity);
    rays_in ri{rays->ox, rays->oy, rays->oz, rays->dx, rays->dy, rays->dz, rays->tmax, rays->pix};
    rays_out ro{sorted->ox, sorted->oy, sorted->oz, sorted->dx, sorted->dy, sorted->dz, sorted->tmax, sorted->pix};
    uint32_t cap = rays->capacity;
    nodes_dev nd{nodes->cx, nodes->cy, nodes->cz, nodes->r, nodes->ax, nodes->ay, nodes->az,
                 nodes->c, nodes->s, nodes->tan, nodes->sec, nodes->capacity};
    // launch bounds from the capacity (every frame may add one partial node
    // per level); kernels read the real counts from meta
    const uint64_t extra = bd ? bd->n_frames : 0;
    uint64_t cnt = ((uint64_t)cap + bundle - 1) / bundle + extra;
    uint32_t g;
    {
        prof_scope ps("k_build_leaf", stream), pp("k_permute", stream);
#define CRSH_LEAF(NB)                                                                                      \
    (g = (uint32_t)std::max<uint64_t>((cnt + LEAF_RAYS / NB - 1) / (LEAF_RAYS / NB), 1),                   \
     bd ? k_build_leaf<NB, true><<<g, LEAF_THREADS, 0, stream>>>(ri, sorted_ids, ro, bundle, merge, levels, nd, meta, \
                                                                 cap, b)                                   \
        : k_build_leaf<NB, false><<<g, LEAF_THREADS, 0, stream>>>(ri, sorted_ids, ro, bundle, merge, levels, nd, meta, \
                                                                  cap, b))
        switch (pow2_at_least(bundle)) {
        case 1: CRSH_LEAF(1); break;
        case 2: CRSH_LEAF(2); break;
        case 4: CRSH_LEAF(4); break;
        case 8: CRSH_LEAF(8); break;
        case 16: CRSH_LEAF(16); break;
        default: CRSH_LEAF(32); break;
        }
#undef CRSH_LEAF
    }
    int nf = pow2_at_least(merge);
#define CRSH_UP(NF)                                                                                        \
    (tail ? (bd ? k_build_tail<NF, true><<<1, UP_TAIL, 0, stream>>>(lv, merge, nd, meta, b)               \
                : k_build_tail<NF, false><<<1, UP_TAIL, 0, stream>>>(lv, merge, nd, meta, b))             \
          : (bd ? k_build_up<NF, true><<<g, 256, 0, stream>>>(lv, merge, nd, meta, b)                     \
                : k_build_up<NF, false><<<g, 256, 0, stream>>>(lv, merge, nd, meta, b)))
    for (int lv = 1; lv < levels; ++lv) {
        cnt = (cnt + merge - 1) / merge + extra;
        // cnt bounds this level, and the ones above it have no more
        const bool tail = cnt <= UP_TAIL;
        g = (uint32_t)std::min<uint64_t>((cnt + 255) / 256, 1u << 22);
        if (g == 0) g = 1;
        switch (nf) {
        case 2: CRSH_UP(2); break;
        case 4: CRSH_UP(4); break;
        case 8: CRSH_UP(8); break;
        default: CRSH_UP(16); break;
        }
        if (tail) break;
    }
#undef CRSH_UP
    return hip_check(hipGetLastError(), "crsh_build launch");
}

}  // namespace crsh

extern "C" crsh_status crsh_build(const crsh_rays *rays, const uint32_t *sorted_ids, int32_t bundle, int32_t merge,
                                  int32_t levels, crsh_nodes *nodes, crsh_rays *sorted, crsh_meta *meta,
                                  hipStream_t stream)
{
    return build_launch(rays, sorted_ids, bundle, merge, levels, nodes, sorted, meta, nullptr, stream);
}
