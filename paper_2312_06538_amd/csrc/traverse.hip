// Stage 4: hierarchy traversal (Sec. 3.3.7, Eq. 9).
//
// A level's pairs are written together with what the next level needs of
// them: the Eq. 9 tests of every pair's children run where the pair is
// emitted, while its triangle and node are in registers.  Per level:
//   scan   exclusive scan of the survivors of every tile of pairs -> where a
//          tile's children go on the next level;
//   step   the pairs of a tile that have surviving children write them at that
//          place, in (parent pair, child) order, staged through LDS; every
//          pair written is tested against the children of its node at once
//          (child nodes read from a run of them copied to LDS) and leaves a
//          pass bit per child and the survivors of its tile for the next scan.
// The top level comes before, from its own count (one (top node, mesh) pair
// per wave), scan and emit; its emit tests the children in the same way.  No
// launch waits between blocks but the scan's look-back.
// The pair arrays come out trimmed (Fig. 4) and in the order of a sequential
// traversal, so they are deterministic.  Pairs are two arrays (triangle, node)
// or, for crsh_traverse_packed, one 32-bit word each (Sec. 3.3.7's encoding),
// a compile-time choice of every kernel.
//
// Batched form: frames have their own top levels, so levels are produced from
// the highest down; on each level the pairs that descend from the level above
// come first, then a top-level pass appends the (node, mesh, triangle) pairs
// of the frames whose top is this level.  A top-level item is (frame, top
// node, mesh of the frame); a parent's children are the range recorded with
// it by the build (first child, count), so below the top a frame is looked
// up only when a block copies a new run of child nodes to LDS.
//
// crsh_leaf_hit forms the level-1 pass bits from the stored level-2 pairs with
// a count pass of its own (k_level_count_lanes).
#include "bounds.hpp"
#include "traverse.hpp"


namespace crsh {

// One launch before the traversal:
// - bounding spheres of the triangles [b, e);
// - traversal copy of the nodes: (cx, cy, cz, r), (ax, ay, az, tan) and sec,
//   with sec = -1 marking a cone of 90 degrees or more (c <= 0 gives no
//   positive sec, c > 0 always does), so one test reads 36 bytes in 3 loads;
// - n_cnt tile counts and the workgroup sums of S cleared (n_cnt != 0), the
//   per-call pair counts cleared and a hierarchy of more levels than there is
//   pair storage for flagged (levels != 0).
__global__ void k_trav_prep(tri_verts V, uint32_t b, uint32_t e, float4 *tsph, node_arrays nd, crsh_meta *meta,
                            float4 *na, float4 *nb, float *ns, trav_scratch S, uint64_t n_cnt, uint32_t levels)
{
    const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    const uint32_t nl = meta->n_levels;
    if (levels && gid < CRSH_MAX_LEVELS) meta->pairs[gid] = 0;
    if (levels && gid == 0 && nl > levels) atomicOr(&meta->status, CRSH_OVERFLOW_PAIRS);
    for (uint64_t i = gid; i < n_cnt; i += stride) S.cnt[i] = 0u;
    if (n_cnt && gid < TRAV_PARTS) S.part[gid] = 0u;
    const uint32_t total = nl ? meta->level_off[nl - 1] + meta->level_cnt[nl - 1] : 0;
    for (uint32_t i = gid; i < total; i += stride) {
        na[i] = make_float4(nd.cx[i], nd.cy[i], nd.cz[i], nd.r[i]);
        nb[i] = make_float4(nd.ax[i], nd.ay[i], nd.az[i], nd.tan[i]);
        ns[i] = nd.c[i] > 0.0f ? nd.sec[i] : -1.0f;
    }
    const float third = 1.0f / 3.0f;
    for (uint64_t t = (uint64_t)b + gid; t < e; t += stride) {
        const f3 p = mk(V.v[0][t], V.v[1][t], V.v[2][t]);
        const f3 q = mk(V.v[3][t], V.v[4][t], V.v[5][t]);
        const f3 u = mk(V.v[6][t], V.v[7][t], V.v[8][t]);
        const f3 c = ((p + q) + u) * third;
        float r = fmax2(fmax2(len(p - c), len(q - c)), len(u - c));
        const float m = fmax2(fmax2(fabsf(c.x), fabsf(c.y)), fabsf(c.z));
        r = r + SPHERE_PAD * (r + m);
        tsph[t] = make_float4(c.x, c.y, c.z, r);
    }
}

// Parts that a top-level (node, mesh) item is cut into, its triangles in equal
// shares: an item of 1,280 triangles takes a wave 20 steps of about 1.5 us
// each, and a 128x72 frame has 6 items (top emit 32 us; 9 us in 16 parts).
// Up to 1,024 items, a wave per SIMD (with 4,096 the scan over them and the
// look-ups cost a 128x128 frame 6 us more than the parts save it).  Above
// 4,096 items, of which a wave then has several and most have nothing to test,
// up to 4 parts (`many`) even out the waves: top count, emit and scan 470 to 405
// us on 512x512 reflections of 262,144 items, 866 to 815 on a 1080p frame; 2
// parts 402 and 834, 8 parts 505 and 886.  That holds for meshes of many steps
// (1,240 and 1,880 triangles on average there).  Smaller ones gain nothing, and
// every part looks its item up and adds to the count of a tile that many others
// add to: traversals of 512x512 shadow rays against meshes of 233 triangles on
// average (180,224 items) 164 us in one part, 316 in four, of 931 (180,224 items)
// 206 and 337, of 931 (90,112) 161 and 184, of 1,116 (94,208) 157 and 151.  So
// four parts from a mean of 1,024 triangles (top_many).  Between 1,025 and 4,096
// items, one to four for a wave, one part each (not measured there).
__device__ __forceinline__ uint32_t top_parts(uint64_t items, uint64_t cap, uint32_t many)
{
    uint32_t s = 1;
    const uint64_t lim = items > 4096 ? many * items : 1024u;
    while (s < 16 && items * s * 2 <= lim && items * s * 2 <= cap) s *= 2;
    return s;
}

static uint32_t top_many(uint32_t m, uint32_t n_mesh)
{
    const uint32_t mean = m / std::max(n_mesh, 1u);
    return mean >= 1024u ? 4u : 1u;
}

// number of work items of a level: top level (parent_level 0) = top nodes x
// meshes x parts (top_parts), lower levels = tiles of `tile` parent pairs
__device__ __forceinline__ uint64_t level_items(const crsh_meta *meta, int32_t parent_level, uint32_t n_mesh,
                                                const pair_levels &P, uint32_t tile, uint64_t top_cap,
                                                uint32_t many, uint32_t &parts)
{
    const uint32_t nl = meta->n_levels;
    parts = 1;
    if (parent_level == 0) {
        const uint64_t items = nl ? (uint64_t)meta->level_cnt[nl - 1] * n_mesh : 0;
        parts = top_parts(items, top_cap, many);
        return items * parts;
    }
    if ((uint32_t)parent_level > nl || parent_level < 2) return 0;
    uint64_t nin = meta->pairs[parent_level - 1];
    const uint64_t cap = P.p[parent_level - 1].cap;
    nin = nin < cap ? nin : cap;
    return (nin + tile - 1) / tile;
}

// the look-back words and the ticket of the scan that follows this launch
__device__ __forceinline__ void clear_scan(const trav_scratch &S)
{
    const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
    for (uint32_t i = gid; i < S.n_flags; i += gridDim.x * blockDim.x) S.scan_flags[i] = 0;
    if (gid == 0) *S.scan_ctr = 0;
}

// ------------------------------------------------------------- top level
// Item -> (node i within the level, mesh m).  Plain: item = i * n_mesh + m.
// Batch: the item's frame, then (top node, mesh) within the frame.  A wave's
// items -- wave, wave + nwaves, wave + 2 nwaves, ... -- are looked up one per
// lane, 64 at a time, and those with triangles to test worked on one after
// the other by the whole wave, their values taken from the lane that has
// them.
template <bool BATCH>
__device__ __forceinline__ void top_item(uint64_t item_part, uint32_t parts, uint32_t n_mesh, uint32_t top, uint32_t off,
                                         const batch_dev &bd, const float4 *na, const float4 *nb, const float *ns,
                                         const float *msph, const uint32_t *mesh_first, const uint32_t *mesh_count,
                                         uint32_t tri_begin, uint32_t tri_end, float4 &A, float4 &Bv, float &S,
                                         uint32_t &i, uint32_t &b, uint32_t &e, bool &pass)
{
    uint32_t m;
    const uint64_t item = item_part / parts;
    if constexpr (BATCH) {
        const uint32_t f = frame_of_item(bd, item);
        const uint64_t local = item - bd.fm[f].item_base;
        const uint32_t mc = bd.frames[f].mesh_count;
        const uint32_t li = (uint32_t)(local / mc);
        i = bd.fm[f].level_base[top] + li;
        m = bd.frames[f].mesh_begin + (uint32_t)(local - (uint64_t)li * mc);
    } else {
        i = (uint32_t)item / n_mesh;
        m = (uint32_t)item - i * n_mesh;
    }
    A = na[off + i];
    Bv = nb[off + i];
    S = ns[off + i];
    const bool real = !BATCH || m < n_mesh;    // frames name meshes of the batch's scene
    if (!real) m = 0;
    pass = real && packed_meets(A, Bv, S, mk(msph[4 * m], msph[4 * m + 1], msph[4 * m + 2]), msph[4 * m + 3]);
    b = e = 0;
    if (pass) {
        b = max(mesh_first[m], tri_begin);
        e = min(mesh_first[m] + mesh_count[m], tri_end);
        if (e < b) e = b;
        const uint32_t part = (uint32_t)(item_part - item * parts), n = e - b;
        e = b + (uint32_t)((uint64_t)n * (part + 1) / parts);
        b += (uint32_t)((uint64_t)n * part / parts);
    }
}

__device__ __forceinline__ uint32_t from_lane(uint32_t v, uint32_t src) { return __builtin_amdgcn_readlane(v, src); }
__device__ __forceinline__ float from_lane(float v, uint32_t src)
{
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), src));
}
__device__ __forceinline__ float4 from_lane(float4 v, uint32_t src)
{
    return make_float4(from_lane(v.x, src), from_lane(v.y, src), from_lane(v.z, src), from_lane(v.w, src));
}
__device__ __forceinline__ uint64_t from_lane(uint64_t v, uint32_t src)
{
    return (uint64_t)from_lane((uint32_t)(v >> 32), src) << 32 | from_lane((uint32_t)v, src);
}

// top level of this pass (0-based) and its number of items
template <bool BATCH>
__device__ __forceinline__ bool top_pass(const crsh_meta *meta, const batch_dev &bd, uint32_t L, uint32_t n_mesh,
                                         const pair_levels &P, const trav_scratch &S, uint32_t &top, uint64_t &n_items,
                                         uint32_t &parts)
{
    const uint32_t nl = meta->n_levels;
    if (nl == 0) return false;
    if constexpr (BATCH) {
        if (L > nl) return false;
        top = L - 1;
        n_items = bd.top[0];
        parts = (uint32_t)bd.top[2];
    } else {
        top = nl - 1;
        n_items = level_items(meta, 0, n_mesh, P, 1u, S.top_cap, S.top_many, parts);
    }
    return true;
}

template <bool BATCH>
__global__ __launch_bounds__(256) void k_top_count(const float4 *__restrict__ na, const float4 *__restrict__ nb,
                                                   const float *__restrict__ ns, const float4 *__restrict__ tsph,
                                                   const uint32_t *__restrict__ mesh_first,
                                                   const uint32_t *__restrict__ mesh_count,
                                                   const float *__restrict__ msph, uint32_t n_mesh,
                                                   uint32_t tri_begin, uint32_t tri_end, pair_levels P,
                                                   trav_scratch S, crsh_meta *meta, batch_dev bd, uint32_t L)
{
    __shared__ uint64_t s_red[3][256 / WAVE];
    uint32_t top, parts;
    uint64_t n_items;
    clear_scan(S);
    if (!top_pass<BATCH>(meta, bd, L, n_mesh, P, S, top, n_items, parts)) return;
    const uint32_t off = meta->level_off[top];
    const uint32_t l = lane_id();
    const uint64_t wave = (uint64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE;
    const uint64_t nwaves = (uint64_t)gridDim.x * (blockDim.x / WAVE);
    uint64_t tests = 0, mhits = 0, items = 0;       // tests: this lane's
    for (uint64_t it0 = wave; it0 < n_items; it0 += nwaves * WAVE) {
        const uint64_t it = it0 + l * nwaves;
        const bool real = it < n_items;
        float4 lA, lB;
        float lS;
        uint32_t i, lb, le;
        bool pass;
        top_item<BATCH>(real ? it : it0, parts, n_mesh, top, off, bd, na, nb, ns, msph, mesh_first, mesh_count, tri_begin,
                        tri_end, lA, lB, lS, i, lb, le, pass);
        const bool whole = real && it % parts == 0;     // an item counts with its first part
        items += (uint64_t)__popcll(ballot(whole));
        mhits += (uint64_t)__popcll(ballot(whole && pass));
        if (real) tests += le - lb;
        if (real && le == lb) S.cnt_top[it] = 0u;
        for (uint64_t todo = ballot(real && le > lb); todo; todo &= todo - 1u) {
            const uint32_t src = (uint32_t)__builtin_ctzll(todo);
            const float4 A = from_lane(lA, src), Bv = from_lane(lB, src);
            const float Sg = from_lane(lS, src);
            const uint32_t b = from_lane(lb, src), e = from_lane(le, src);
            uint32_t cnt = 0;
            for (uint32_t t0 = b; t0 < e; t0 += WAVE) {
                const uint32_t t = t0 + l;
                bool ok = false;
                if (t < e) {
                    const float4 s = tsph[t];
                    ok = packed_meets(A, Bv, Sg, mk(s.x, s.y, s.z), s.w);
                }
                cnt += (uint32_t)__popcll(ballot(ok));
            }
            if (l == src) S.cnt_top[it] = cnt;
        }
    }
    tests = wave_sum(tests);
    if (l == 0) {
        s_red[0][threadIdx.x / WAVE] = tests;
        s_red[1][threadIdx.x / WAVE] = mhits;
        s_red[2][threadIdx.x / WAVE] = items;
    }
    // the scan that follows adds the blocks' sums to meta (atomics of every
    // block on three words would outlast a small frame's pass)
    __syncthreads();
    if (threadIdx.x < 3) {
        uint64_t t = 0;
        for (int w = 0; w < 256 / WAVE; ++w) t += s_red[threadIdx.x][w];
        S.top_part[3 * blockIdx.x + threadIdx.x] = t;
    }
}

// Pass bits of a pair's children: one byte per pair for merge factors up to
// 8, else two.
template <int NF>
struct mask_type {
    typedef uint8_t t;
};
template <>
struct mask_type<16> {
    typedef uint16_t t;
};

// Many items of small meshes come TOP_RUN at a time to a wave, neighbours in the
// pair list, so that their survivors, most of one tile, are added to its count at
// once: traversal of 512x512 shadow rays, 180,224 items, 165 us one by one, 118
// in twos, 100 in fours, 104 in eights (larger meshes, 206, 160, 169, 210).  Not those
// of larger meshes that have one part for want of item storage: 128x72 mixed rays,
// one level, 178 us one by one, 230 in fours.
constexpr uint32_t TOP_RUN = 4;

// NF: the merge factor rounded up to a power of two.  Top-level pairs written
// at or above level `lowest` + 1 are tested against their node's children.
template <int NF, bool BATCH, bool PACKED>
__global__ __launch_bounds__(256) void k_top_emit(const float4 *__restrict__ na, const float4 *__restrict__ nb,
                                                  const float *__restrict__ ns, const float4 *__restrict__ tsph,
                                                  const uint32_t *__restrict__ mesh_first,
                                                  const uint32_t *__restrict__ mesh_count,
                                                  const float *__restrict__ msph, uint32_t n_mesh,
                                                  uint32_t tri_begin, uint32_t tri_end, uint32_t F, uint32_t lowest,
                                                  pair_levels P, trav_scratch S, const crsh_meta *meta, batch_dev bd,
                                                  uint32_t L)
{
    typedef typename mask_type<NF>::t mask_t;
    constexpr uint32_t TILE = step_tile(NF);
    __shared__ uint64_t s_red[256 / WAVE];
    __shared__ float4 s_ca[256 / WAVE][NF], s_cb[256 / WAVE][NF];   // a wave's item: children of its node
    __shared__ float s_cs[256 / WAVE][NF];
    const uint32_t wib = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    uint32_t top, parts;
    uint64_t n_items;
    clear_scan(S);
    if (!top_pass<BATCH>(meta, bd, L, n_mesh, P, S, top, n_items, parts)) return;
    const pairs_dev out = P.p[top];
    if (out.tri == nullptr) return;
    const bool test = top >= lowest;         // level top + 1 (1-based) >= lowest + 1
    mask_t *const mask = (mask_t *)S.mask[(top + 1) & 1];
    const uint32_t off = meta->level_off[top];
    const uint32_t offk = test ? meta->level_off[top - 1] : 0u, nk = test ? meta->level_cnt[top - 1] : 0u;
    const uint32_t l = lane_id();
    const uint64_t wave = (uint64_t)blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE;
    const uint64_t nwaves = (uint64_t)gridDim.x * (blockDim.x / WAVE);
    uint64_t tests = 0;
    const uint64_t run = S.top_many == 1 && parts == 1 && n_items > 4096 ? TOP_RUN : 1u;
    const uint64_t lane_it = l / run * nwaves * run + l % run;
    for (uint64_t it0 = wave * run; it0 < n_items; it0 += nwaves * WAVE) {
        const uint64_t it = it0 + lane_it;
        const bool some = it < n_items && S.cnt_top[it] != 0;
        uint64_t todo = ballot(some);
        if (todo == 0) continue;
        float4 lA, lB;
        float lS;
        uint32_t li, lb, le;
        bool pass;
        const uint32_t one = (uint32_t)__builtin_ctzll(todo);
        const uint64_t use = some ? it : it0 + one / run * nwaves * run + one % run;
        top_item<BATCH>(use, parts, n_mesh, top, off, bd, na, nb, ns, msph, mesh_first, mesh_count, tri_begin, tri_end,
                        lA, lB, lS, li, lb, le, pass);
        const uint64_t lpos = S.off[use];
        // the node's children
        uint32_t lfirst = li * F, lnch = 0u;
        if (test) {
            lnch = lfirst < nk ? min(F, nk - lfirst) : 0u;
            if constexpr (BATCH) {
                lfirst = bd.node_first[off + li];
                lnch = lfirst < nk ? min(bd.node_info[off + li] & INFO_COUNT_MASK, nk - lfirst) : 0u;
            }
        }
        uint64_t tile = 0;                       // tile being written, and its survivors so far
        uint32_t in_tile = 0u;
        for (; todo; todo &= todo - 1u) {
            const uint32_t src = (uint32_t)__builtin_ctzll(todo);
            const float4 A = from_lane(lA, src), Bv = from_lane(lB, src);
            const float Sg = from_lane(lS, src);
            const uint32_t i = from_lane(li, src), b = from_lane(lb, src), e = from_lane(le, src);
            const uint32_t first = from_lane(lfirst, src), nch = from_lane(lnch, src);
            __builtin_amdgcn_wave_barrier();     // the previous item's reads come first
            if (l < nch) {
                s_ca[wib][l] = na[offk + first + l];
                s_cb[wib][l] = nb[offk + first + l];
                s_cs[wib][l] = ns[offk + first + l];
            }
            __builtin_amdgcn_wave_barrier();
            uint64_t pos = from_lane(lpos, src);
            if (pos / TILE != tile) {
                if (l == 0 && in_tile) atomicAdd(&S.cnt[tile], in_tile);
                tile = pos / TILE;
                in_tile = 0u;
            }
            float4 s_n = b < e ? tsph[min(b + l, e - 1)] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            for (uint32_t t0 = b; t0 < e; t0 += WAVE) {
                const uint32_t t = t0 + l;
                const float4 s = s_n;                // the next 64 are requested before these are tested
                s_n = tsph[min(min(t0 + WAVE, e - 1) + l, e - 1)];
                const uint64_t in_mesh = e - t0 >= WAVE ? ~0ull : (1ull << (e - t0)) - 1ull;
                const uint64_t mk64 = packed_meets_mask(A, Bv, Sg, mk(s.x, s.y, s.z), s.w) & in_mesh;
                if (mk64 == 0) continue;
                const uint32_t rank = rank_below(mk64);
                const uint64_t at = pos + rank;
                const bool put = ((mk64 >> l) & 1u) && at < out.cap;
                if (put) pair_put<PACKED>(out, at, t, i);
                if (test) {
                    const uint64_t pm = ballot(put);
                    // the lanes whose pair lies in the current tile; the others in the next
                    const uint64_t in = ballot(at / TILE == tile);
                    uint32_t bits = 0u, ca = 0u, cb = 0u;
                    auto child = [&](uint32_t r) {
                        const uint64_t m = packed_meets_mask(s_ca[wib][r], s_cb[wib][r], s_cs[wib][r],
                                                             mk(s.x, s.y, s.z), s.w) & pm;
                        bits = bits + bits + (__builtin_amdgcn_inverse_ballot_w64(m) ? 1u : 0u);
                        ca += (uint32_t)__popcll(m & in);
                        cb += (uint32_t)__popcll(m & ~in);
                    };
                    if (nch == NF) {
#pragma unroll
                        for (uint32_t r = NF; r-- > 0;) child(r);
                    } else {
                        for (uint32_t r = nch; r-- > 0;) child(r);
                    }
                    if (put) mask[at] = (mask_t)bits;
                    tests += (uint64_t)__popcll(pm) * nch;
                    in_tile += ca;
                    if ((pos + (uint32_t)__popcll(mk64)) / TILE != tile) {
                        if (l == 0 && in_tile) atomicAdd(&S.cnt[tile], in_tile);
                        ++tile;
                        in_tile = cb;
                    }
                }
                pos += (uint32_t)__popcll(mk64);
            }
        }
        if (l == 0 && in_tile) atomicAdd(&S.cnt[tile], in_tile);
    }
    if (l == 0) s_red[threadIdx.x / WAVE] = tests;
    __syncthreads();
    if (threadIdx.x == 0) S.part[blockIdx.x] += s_red[0] + s_red[1] + s_red[2] + s_red[3];
}

// ----------------------------------------------------------- lower levels
// Lane i of each quad of four lanes gets the value of lane (i / NF) * NF + r
// of its quad (NF <= 4: the NF lanes of a group share one source lane).  r
// is a constant once the slice loop is unrolled; the switch folds away.
template <uint32_t NF>
__device__ __forceinline__ uint32_t quad_pick(uint32_t v, uint32_t r)
{
    static_assert(NF == 2 || NF == 4, "groups within a quad");
#define CRSH_QP(R) ((((0 / NF) * NF + (R)) & 3) | ((((1 / NF) * NF + (R)) & 3) << 2) | \
                    ((((2 / NF) * NF + (R)) & 3) << 4) | ((((3 / NF) * NF + (R)) & 3) << 6))
    switch (r) {
    case 0: return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CRSH_QP(0), 0xF, 0xF, true);
    case 1: return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CRSH_QP(1), 0xF, 0xF, true);
    case 2: return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CRSH_QP(2), 0xF, 0xF, true);
    default: return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CRSH_QP(3), 0xF, 0xF, true);
    }
#undef CRSH_QP
}
template <uint32_t NF>
__device__ __forceinline__ float quad_pick(float v, uint32_t r)
{
    return __uint_as_float(quad_pick<NF>(__float_as_uint(v), r));
}
// The same through the other DPP builtin: a second, separate copy of a value
// quad_pick already took (the compiler folds a DPP move into the one
// instruction that uses it, and would merge two identical moves).
template <uint32_t NF>
__device__ __forceinline__ float quad_pick_again(float v, uint32_t r)
{
#define CRSH_QP(R) ((((0 / NF) * NF + (R)) & 3) | ((((1 / NF) * NF + (R)) & 3) << 2) | \
                    ((((2 / NF) * NF + (R)) & 3) << 4) | ((((3 / NF) * NF + (R)) & 3) << 6))
    const int x = (int)__float_as_uint(v);
    switch (r) {
    case 0: return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, x, CRSH_QP(0), 0xF, 0xF, true));
    case 1: return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, x, CRSH_QP(1), 0xF, 0xF, true));
    case 2: return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, x, CRSH_QP(2), 0xF, 0xF, true));
    default: return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, x, CRSH_QP(3), 0xF, 0xF, true));
    }
#undef CRSH_QP
}

// Count pass with one (parent pair, child) test per lane.
// A tile of LEVEL_TILE parent pairs is tested in NF slices of LEVEL_TILE /
// NF parents; in a slice the NF lanes of a parent test its NF consecutive
// children, and the wave's ballot is directly the pass bits of its 64 / NF
// parents in the mask layout of the count pass (NF bits per parent,
// parent-major).  A block of COUNT_THREADS takes COUNT_TPS tiles per step.
// What the NF lanes of a parent share -- the parent's children and the
// triangle sphere -- is read once: each lane reads the pair and sphere of
// one of the wave's 64 parents of the tile.  For NF <= 4 that lane is one
// of the parent's NF lanes (lane NF * p + r holds parent p of slice r), and
// in slice r the others take the values from it within their quad of lanes
// (a DPP broadcast, no LDS); for larger NF the lanes put them in a
// wave-private LDS record and the lanes of a slice read their parent's
// record from there.  The next step's pairs and spheres are requested
// before a step is tested (pairs two steps ahead, since the sphere read
// depends on them).
//
// Child nodes (36 bytes a test) come from LDS where they can: the
// descendants of one top-level node on the child level are a contiguous
// run of F^(levels above the child level) nodes, aligned to that length
// from the frame's first node of the level, and the pairs of a level are
// ordered by top-level node first, so a block's consecutive steps keep
// testing children from the same run.  When the run fits COUNT_WINDOW
// nodes, the block copies the run holding its step's first child, and the
// runs after it as far as the window reaches within the frame, into LDS
// (once per window it enters; the batched form looks the frame up only
// then) and its waves read the children there; a group of slices with a
// child outside the window reads the node arrays directly.  In the batched form a
// parent's children are the range the build recorded with it (first,
// count); the lane that reads a parent's pair reads that record too, in the
// same stage as the sphere, and puts it in the parent's LDS record.
template <int NF, bool BATCH, bool STAGED>
__global__ __launch_bounds__(COUNT_THREADS) void k_level_count_lanes(int32_t parent_level, uint32_t F,
                                                                     const float4 *__restrict__ na,
                                                                     const float4 *__restrict__ nb,
                                                                     const float *__restrict__ ns,
                                                                     const float4 *__restrict__ tsph, uint32_t m,
                                                                     pair_levels P, trav_scratch S, crsh_meta *meta,
                                                                     batch_dev bd)
{
    static_assert(LEVEL_PPT == 1 && WAVE % NF == 0, "whole parents per wave");
    constexpr uint32_t PR = LEVEL_THREADS / NF;   // parents per slice; NF slices make a tile
    constexpr uint32_t PW = WAVE / NF;            // parents of a wave per slice
    constexpr uint32_t WPT = LEVEL_THREADS / WAVE;   // waves per tile
    constexpr uint32_t NW = COUNT_THREADS / WAVE;    // waves per block
    constexpr uint32_t NONE = 0xFFFFFFFFu;
    constexpr uint32_t WN = STAGED ? COUNT_WINDOW : 1u;
    constexpr bool QB = NF <= 4;             // parent values by quad broadcast
    constexpr uint32_t NR = QB ? 1u : NW;    // wave records in LDS
    __shared__ uint32_t s_red32[2][NW];
    __shared__ uint64_t s_red[NW];
    __shared__ uint32_t s_head[2];          // the step's first pair: 16 x (first child, children)
    __shared__ float4 s_sph[NR][WAVE];      // [wave][record]
    __shared__ uint32_t s_first[NR][WAVE];  // 16 x first child (level-local)
    __shared__ uint32_t s_n[NR][WAVE];      // 16 x children below nk (0: none)
    __shared__ float4 s_wa[WN], s_wb[WN];   // the staged run of child nodes
    __shared__ float s_ws[WN];
    const uint32_t nl = meta->n_levels;
    if ((uint32_t)parent_level > nl || parent_level < 2) return;
    uint32_t parts;
    const uint64_t ntiles = level_items(meta, parent_level, 0, P, LEVEL_TILE, 0, 1u, parts);
    const pairs_dev in = P.p[parent_level - 1];
    if (in.tri == nullptr || P.p[parent_level - 2].tri == nullptr) return;
    uint64_t nin = meta->pairs[parent_level - 1];
    nin = nin < in.cap ? nin : in.cap;
    const uint64_t nsteps = (ntiles + COUNT_TPS - 1) / COUNT_TPS;
    const uint32_t nk = meta->level_cnt[parent_level - 2];
    const uint32_t offk = meta->level_off[parent_level - 2];
    const uint32_t offp = meta->level_off[parent_level - 1];
    const uint32_t np = meta->level_cnt[parent_level - 1];
    const uint32_t F16 = F * 16u, nk16 = nk * 16u;
    const uint32_t l = lane_id();
    // wave indices, made scalar so that the addresses built from them are
    // scalar arithmetic
    const uint32_t wb = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);   // wave of the block
    const uint32_t half = wb / WPT;                   // tile of the step
    const uint32_t tw = wb % WPT;                     // wave of the tile
    const uint32_t j = l % NF;              // child of this lane in every slice
    const uint32_t j16 = j * 16u;
    const uint32_t mlane = l == 0 ? 0u : 0x80000000u;   // mask stores: past the range but for lane 0
    const uint32_t pi = l / NF;             // parent of this lane within the wave's slice
    // the parent whose pair and sphere this lane reads: quad broadcast,
    // slice j, parent pi of the wave's share of it; else slice l / PW,
    // parent l % PW
    const uint32_t own = QB ? j * PR + tw * PW + pi : (l / PW) * PR + tw * PW + l % PW;
    // nodes from offk + ch for ch < nk, by 32-bit byte offsets
    const uint64_t nodes = (uint64_t)offk + nk;
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(na, nodes * 16u);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(nb, nodes * 16u);
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(ns, nodes * 4u);
    // descendants of one top-level node on the child level of a hierarchy
    // with `levels` levels: F^(levels - L + 1) (above WN: more than the
    // window holds)
    auto run_of = [&](uint32_t levels) {
        uint32_t run = 1;
        for (uint32_t e = 0; e < levels - (uint32_t)parent_level + 1 && run <= WN; ++e) run *= F;
        return run;
    };
    // STAGED: the host's bound on the runs of this level fits the window
    const bool staged = STAGED && (BATCH || run_of(nl) <= WN);
    uint32_t wlo = NONE, wlen = 0;          // staged run (block-uniform)
    uint32_t wlo16 = 0u, wlen16 = 0u;       // the same, x 16
    uint32_t ulo = NONE, ulen = 0;          // batch: a frame's nodes whose runs do not fit
    // the pair this lane reads for a step, by buffer loads over the tile's
    // pairs (a step past the end reads nothing): no branch, so that the
    // loads of every step count alike where the compiler places its waits
    auto load_pair = [&](uint64_t step, uint32_t &tri, uint32_t &par) {
        const uint64_t q0 = (step * COUNT_TPS + half) * LEVEL_TILE;
        // pairs of the tile: min(nin - q0, LEVEL_TILE), 0 past the end, in
        // 32-bit scalar operations (both below 2^63)
        const uint64_t left = nin - q0;
        const uint32_t lhi = (uint32_t)(left >> 32), llo = (uint32_t)left;
        const uint32_t nq = lhi == 0u ? min(llo, (uint32_t)LEVEL_TILE) : (lhi >> 31 ? 0u : (uint32_t)LEVEL_TILE);
        const __amdgpu_buffer_rsrc_t rt = make_rsrc(in.tri + q0, (uint64_t)nq * 4u);
        const uint32_t w = __builtin_amdgcn_raw_buffer_load_b32(rt, own * 4u, 0, 0);
        const __amdgpu_buffer_rsrc_t rn = make_rsrc(in.node + q0, (uint64_t)nq * 4u);
        tri = w;
        par = own < nq ? __builtin_amdgcn_raw_buffer_load_b32(rn, own * 4u, 0, 0) : NONE;
    };
    uint64_t tests = 0;                     // wave-wide
    uint32_t parity = 0;
    // a parent's children: plain, par * F + [0, F); batch, the build's
    // record (level-local first child, count); as 16 x (first, number below
    // nk), byte offsets into the staged run (node indices stay below 2^28:
    // 32-bit byte offsets into the node arrays)
    auto children = [&](uint32_t par, uint32_t &first16, uint32_t &n16) {
        if constexpr (BATCH) {
            const bool ok = par < np;
            const uint32_t first = ok ? bd.node_first[offp + par] : 0u;
            const uint32_t cnt = ok ? bd.node_info[offp + par] & INFO_COUNT_MASK : 0u;
            first16 = first < nk ? first * 16u : 0u;
            n16 = first < nk ? (min(first + cnt, nk) - first) * 16u : 0u;
        } else {
            // a parent below np has its first child below nk; F16, nk16:
            // F and nk times 16 (scalar); first16 of no parent is never read
            first16 = par * F16;
            n16 = par < np ? min(F16, nk16 - first16) : 0u;
        }
    };
    // two-stage prefetch: the sphere (and batch: the child range) of the
    // next step and the pair of the step after it are in flight while a
    // step is tested
    uint32_t first_n = 0u, n_n = 0u, tri_nn = 0u, par_nn = NONE;
    float4 sp_n = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (blockIdx.x < nsteps) {
        uint32_t tri0, par0;
        load_pair(blockIdx.x, tri0, par0);
        sp_n = tsph[tri0 < m ? tri0 : 0u];
        children(par0, first_n, n_n);
        load_pair(blockIdx.x + gridDim.x, tri_nn, par_nn);
    }
    // the prologue's loads are in before the loop: the waits the compiler
    // places in the loop then count only the loop's own memory operations
    // (not every store of the previous step)
    __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0)
    // a 32-bit step index (steps stay far below 2^31: 512 pairs a step), so
    // the loop's bookkeeping is scalar arithmetic
    const uint32_t nsteps32 = (uint32_t)min(nsteps, (uint64_t)0x7FFFFFFFu);
    for (uint32_t step = blockIdx.x; step < nsteps32; step += gridDim.x, parity ^= 1u) {
        const uint64_t tile = step * COUNT_TPS + half;
        // this wave's slice-0 word of the tile's pass masks (scalar)
        uint2 *const mrow = (uint2 *)S.bits + (tile * LEVEL_TILE + tw * PW) * NF / 64;
        const __amdgpu_buffer_rsrc_t mrs = make_rsrc(mrow, tile < ntiles ? (NF - 1) * (PR * NF / 64) * 8u + 8u : 0u);
        // this step's parent values: kept in registers (quad broadcast) or
        // put in the wave's records (the wave's previous reads of them are
        // done: program order within the wave); the step's first pair is
        // lane 0's of wave 0
        const float4 sp_c = sp_n;
        const uint32_t first_c = first_n, n_c = n_n;
        if constexpr (!QB) {
            __builtin_amdgcn_wave_barrier();
            s_sph[wb][l] = sp_n;
            s_first[wb][l] = first_n;
            s_n[wb][l] = n_n;
            __builtin_amdgcn_wave_barrier();
        }
        if (staged && wb == 0 && l == 0) {
            s_head[0] = first_n;
            s_head[1] = n_n;
        }
        if (staged) {
            // every wave has finished its reads of the staged run (they
            // precede the previous step's count barrier)
            __syncthreads();
            const uint32_t c0 = s_head[0] / 16u;
            if (s_head[1] != 0u && c0 - wlo >= wlen && c0 - ulo >= ulen) {
                // the frame's nodes on the child level and its levels
                uint32_t base = 0u, cntf = nk, levels = nl;
                if constexpr (BATCH) {
                    const uint32_t f = frame_of_node(bd, (uint32_t)parent_level - 2, c0);
                    base = bd.fm[f].level_base[parent_level - 2];
                    cntf = bd.fm[f].level_cnt[parent_level - 2];
                    levels = bd.fm[f].n_levels;
                }
                const uint32_t run = run_of(levels);
                if (run <= WN && c0 >= base && c0 - base < cntf) {
                    // as many whole runs as the window holds, from the one
                    // holding c0 (later steps move on to the next runs)
                    const uint32_t lo = base + (c0 - base) / run * run;
                    const uint32_t len = min(WN / run * run, base + cntf - lo);
                    for (uint32_t i = threadIdx.x; i < len; i += COUNT_THREADS) {
                        s_wa[i] = na[offk + lo + i];
                        s_wb[i] = nb[offk + lo + i];
                        s_ws[i] = ns[offk + lo + i];
                    }
                    __syncthreads();
                    wlo = lo;
                    wlen = len;
                    wlo16 = lo * 16u;
                    wlen16 = len * 16u;
                } else {
                    ulo = base;
                    ulen = cntf;
                }
            }
        }
        sp_n = tsph[tri_nn < m ? tri_nn : 0u];
        children(par_nn, first_n, n_n);
        load_pair(step + 2u * gridDim.x, tri_nn, par_nn);
        uint32_t c = 0;
        // slices in groups of K: every node read of a group is issued before
        // its first test, and the test has no branch to sink them into.
        // Which lanes test a child, and which of those find it outside the
        // staged run, are wave masks (scalar registers), and so are the
        // results; children outside the run are read from the node arrays
        // afterwards, in a branch of their own, so the reads from LDS never
        // wait behind memory loads.
        constexpr uint32_t KG = 2;
        constexpr uint32_t K = NF < KG ? NF : KG;
#pragma unroll
        for (uint32_t r0 = 0; r0 < NF; r0 += K) {
            uint64_t okm[K], outm[K], bal[K];
            uint32_t ch16[K], idx16[K];
            f3 pc[K];                       // the parent's triangle sphere (records)
            float pr[K];
            // the same by quad broadcast, taken where it is used (each copy
            // has one use: the compiler folds it into that instruction)
            auto sph_c = [&](uint32_t k) {
                if constexpr (QB)
                    return mk(quad_pick<NF>(sp_c.x, r0 + k), quad_pick<NF>(sp_c.y, r0 + k), quad_pick<NF>(sp_c.z, r0 + k));
                else
                    return pc[k];
            };
            auto sph_r = [&](uint32_t k) {
                if constexpr (QB)
                    return quad_pick<NF>(sp_c.w, r0 + k);
                else
                    return pr[k];
            };
#pragma unroll
            for (uint32_t k = 0; k < K; ++k) {
                const uint32_t r = r0 + k;
                uint32_t f16, n16;
                if constexpr (QB) {
                    f16 = quad_pick<NF>(first_c, r);
                    n16 = quad_pick<NF>(n_c, r);
                } else {
                    const uint32_t rec = r * PW + pi;
                    f16 = s_first[wb][rec];
                    n16 = s_n[wb][rec];
                    const float4 sp = s_sph[wb][rec];
                    pc[k] = mk(sp.x, sp.y, sp.z);
                    pr[k] = sp.w;
                }
                ch16[k] = f16 + j16;
                okm[k] = ballot(j16 < n16);
                const uint32_t i16 = ch16[k] - wlo16;
                outm[k] = okm[k] & ~ballot(i16 < wlen16);
                // any slot of the window for a lane that tests nothing here
                idx16[k] = min(i16, (WN - 1u) * 16u);
            }
            if constexpr (STAGED) {
                float4 A[K], Bv[K];
                float Sg[K];
#pragma unroll
                for (uint32_t k = 0; k < K; ++k) {
                    A[k] = *(const float4 *)((const char *)s_wa + idx16[k]);
                    Bv[k] = *(const float4 *)((const char *)s_wb + idx16[k]);
                    Sg[k] = *(const float *)((const char *)s_ws + idx16[k] / 4u);
                }
#pragma unroll
                for (uint32_t k = 0; k < K; ++k)
                    bal[k] = packed_meets_mask(A[k], Bv[k], Sg[k], sph_c(k), sph_r(k)) & okm[k] & ~outm[k];
                // rare: a slice with children outside the run, one at a time
                uint64_t any_out = 0;
#pragma unroll
                for (uint32_t k = 0; k < K; ++k) any_out |= outm[k];
                if (any_out != 0) {
#pragma unroll
                    for (uint32_t k = 0; k < K; ++k) {
                        if (outm[k] == 0) continue;
                        const uint32_t g = offk + (((outm[k] >> l) & 1u) ? ch16[k] / 16u : 0u);
                        const float4 Ag = buf_load4(ra, g * 16u);
                        const float4 Bg = buf_load4(rb, g * 16u);
                        const float Sgg = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, g * 4u, 0, 0));
                        f3 c = pc[k];
                        float d = pr[k];
                        if constexpr (QB) {     // copies of its own (see sph_c)
                            c = mk(quad_pick_again<NF>(sp_c.x, r0 + k), quad_pick_again<NF>(sp_c.y, r0 + k),
                                   quad_pick_again<NF>(sp_c.z, r0 + k));
                            d = quad_pick_again<NF>(sp_c.w, r0 + k);
                        }
                        bal[k] |= packed_meets_mask(Ag, Bg, Sgg, c, d) & outm[k];
                    }
                }
            } else {
                // runs longer than the window: every child from the node
                // arrays, the group's loads issued together (outm == okm)
                float4 A[K], Bv[K];
                float Sg[K];
#pragma unroll
                for (uint32_t k = 0; k < K; ++k) {
                    const uint32_t g = offk + (((okm[k] >> l) & 1u) ? ch16[k] / 16u : 0u);
                    A[k] = buf_load4(ra, g * 16u);
                    Bv[k] = buf_load4(rb, g * 16u);
                    Sg[k] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, g * 4u, 0, 0));
                }
#pragma unroll
                for (uint32_t k = 0; k < K; ++k)
                    bal[k] = packed_meets_mask(A[k], Bv[k], Sg[k], sph_c(k), sph_r(k)) & okm[k];
            }
#pragma unroll
            for (uint32_t k = 0; k < K; ++k) {
                const uint32_t r = r0 + k;
                tests += (uint64_t)__popcll(okm[k]);
                // the wave's pass bits of slice r: bit (tile * LEVEL_TILE +
                // r * PR + tw * PW) * NF of the level's masks, a multiple of 64
                // (r * PR * NF = 64 r words' worth of 4 bits: uint2 4 r).
                // Every lane stores, lane 0 in range: no branch around it
                typedef uint32_t v2u __attribute__((ext_vector_type(2)));
                const v2u w = {(uint32_t)bal[k], (uint32_t)(bal[k] >> 32)};
                __builtin_amdgcn_raw_buffer_store_b64(w, mrs, mlane + r * (PR * NF / 64) * 8u, 0, 0);
                c += (uint32_t)__popcll(bal[k]);
            }
        }
        // survivors of each tile: wave sums in alternating LDS slots (one
        // barrier per step)
        if (l == 0) s_red32[parity][wb] = c;
        __syncthreads();
        if (threadIdx.x % LEVEL_THREADS == 0 && tile < ntiles) {
            uint32_t t = 0;
            for (uint32_t ww = 0; ww < WPT; ++ww) t += s_red32[parity][half * WPT + ww];
            S.cnt[tile] = t;
        }
    }
    if (l == 0) s_red[wb] = tests;          // a wave-wide count: the same in every lane
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t tt = 0;
        for (uint32_t ww = 0; ww < NW; ++ww) tt += s_red[ww];
        if (tt) atomicAdd((unsigned long long *)&meta->tests[parent_level - 2], (unsigned long long)tt);
    }
}

// One level step: tiles of step_tile(NF) parent pairs of level parent_level,
// their surviving children written on the level below and, TEST, tested
// against their own children (level parent_level - 2) for the next step.
//
// A thread holds step_ppt(NF) consecutive parents' pass bits; a block scan
// places their survivors, which are listed in LDS (2 bytes: parent of the
// tile, child), so the writing lanes are full and store consecutive pairs
// whatever the bits.  A lane then owns one written pair: its triangle sphere
// is read once for all its children, its pass bits go out as one byte (two
// for merge factors above 8) and the survivors of every 64 consecutive pairs
// are added up as wave masks, then per tile of the next level in LDS.
//
// Child nodes (36 bytes a test) come from LDS where they can (STAGED): the
// descendants of one top-level node on a level are a contiguous run, aligned
// from the frame's first node, and pairs are ordered by top-level node first,
// so consecutive tiles keep testing children of the same nodes.  A block
// copies the children of the run of nodes that its first written pair names,
// and of as many whole runs after it as fit, child r of every node in an
// array of its own (lanes with neighbouring nodes then read neighbouring
// 16 bytes); pairs outside the copy read the node arrays.  Blocks take
// several consecutive tiles at a time where there are enough, so that a copy
// lasts.
//
// Where a top-level node has more descendants than the copy holds (not STAGED)
// every child comes from the node arrays, and lanes work in groups of NF: in
// turn r a group tests the pair of its lane r, a child a lane, so that it reads
// F consecutive nodes (pair and sphere from that lane).  Each lane reading the
// children of its own pair instead, 64 unrelated nodes a load, was bound by the
// vector L1: the step that tests level 1 of 512x512 rays with 4,096 leaves below
// a top node (bundle 4) 6.0 ms with merge factor 8, the traversal 7.2; so 2.7,
// and with merge factor 4 the traversal 4.2 and 2.8.
//
// What bounds it: the tests' arithmetic (1920x1080 frame against 482,048
// triangles, the step that tests level 1: vector issue 81 % busy, 199
// instructions per 64 written pairs, 46 per 64 tests); the last step (no test)
// writes and reads pairs at 4.5 TB/s, near the 5.3 TB/s a large copy reaches.
// Measured on that frame: steps 1.27 + 2.39 + 5.18 + 8.70 + 4.67 ms and the top
// emit 0.59.  A count pass and an emit pass per level, each reading the pair
// list, took 29.0 ms for the traversal of another such frame where the steps take
// 21.1; 1024x1024 reflections 2.07 ms (2.7), 24 frames of a batch 5.3 (7.4).
// Requesting a tile's inputs a tile ahead is what pays for the fusion (24 to 28
// ms without; the next 64 pairs' spheres before these are tested: 21.6 to 21.3
// in all), and 6 waves per SIMD: the compiler's own choice is 4, where only
// merge factors above 8 stay (their lists need the LDS of 4).
template <int NF, bool BATCH, bool PACKED, bool TEST, bool STAGED>
__global__ __launch_bounds__(STEP_THREADS, NF == 16 ? 4 : 6) void k_level_step(int32_t parent_level, uint32_t F,
                                                             const float4 *__restrict__ na,
                                                             const float4 *__restrict__ nb,
                                                             const float *__restrict__ ns,
                                                             const float4 *__restrict__ tsph, uint32_t m,
                                                             pair_levels P, trav_scratch S, const crsh_meta *meta,
                                                             batch_dev bd)
{
    typedef typename mask_type<NF>::t mask_t;
    constexpr uint32_t PPT = step_ppt(NF), TILE = step_tile(NF);
    constexpr uint32_t NW = STEP_THREADS / WAVE;
    constexpr uint32_t WP = COUNT_WINDOW / NF;           // nodes whose children the copy holds
    constexpr uint32_t WN = TEST && STAGED ? COUNT_WINDOW : 1u;
    __shared__ uint16_t s_item[TILE * NF];               // 16 x parent of the tile + child
    __shared__ uint2 s_par[TILE];                        // triangle, first child
    __shared__ uint32_t s_wave[2][NW];
    __shared__ uint32_t s_next[NF + 2];                  // survivors per tile of the next level
    __shared__ float4 s_wa[WN], s_wb[WN];
    __shared__ float s_ws[WN];
    const uint32_t nl = meta->n_levels;
    if (TEST) clear_scan(S);
    if ((uint32_t)parent_level > nl) return;
    const pairs_dev in = P.p[parent_level - 1];
    const pairs_dev out = P.p[parent_level - 2];
    if (in.tri == nullptr || out.tri == nullptr) return;
    uint64_t nin = meta->pairs[parent_level - 1];
    nin = nin < in.cap ? nin : in.cap;
    const uint32_t ntiles = (uint32_t)min((nin + TILE - 1) / TILE, (uint64_t)0x7FFFFFFFu);
    const mask_t *const mask = (const mask_t *)S.mask[parent_level & 1];
    mask_t *const mask_out = (mask_t *)S.mask[(parent_level - 1) & 1];
    const uint32_t offp = meta->level_off[parent_level - 1], np = meta->level_cnt[parent_level - 1];
    // the level written and the level below it
    const uint32_t off1 = meta->level_off[parent_level - 2], n1 = meta->level_cnt[parent_level - 2];
    const uint32_t off2 = TEST ? meta->level_off[parent_level - 3] : 0u;
    const uint32_t n2 = TEST ? meta->level_cnt[parent_level - 3] : 0u;
    const uint32_t l = lane_id();
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    // consecutive tiles of a block: up to 8 where every block gets 8 such shares
    const uint32_t ch = min(max(ntiles / (gridDim.x * 8u), 1u), 8u);
    auto next_of = [&](uint32_t t) { return (t + 1) % ch ? t + 1 : t + 1 + (gridDim.x - 1) * ch; };
    // a tile's inputs: pass bits and pairs of this thread's parents, and the
    // place of the tile's children; nothing looks at them until they are used
    // (`zero` keeps the last a per-lane value: read as a scalar it would be
    // waited for at once), so they arrive while the tile before is worked on.
    // Reads past the level's pairs return zeros (or, one pair past an odd
    // end, bits that are cut off at use).
    uint32_t zero = 0u;
    asm volatile("" : "+v"(zero));
    struct tile_in {
        uint32_t bits, tri[PPT], par[PPT];
        uint64_t off;
    };
    auto load_tile = [&](uint32_t t, tile_in &v) {
        const uint64_t q = (uint64_t)t * TILE;
        const uint32_t n = t < ntiles ? (uint32_t)min(nin - q, (uint64_t)TILE) : 0u;
        const __amdgpu_buffer_rsrc_t rm = make_rsrc(mask + q, ((n + PPT - 1) / PPT) * PPT * (uint32_t)sizeof(mask_t));
        if constexpr (PPT * sizeof(mask_t) == 2)
            v.bits = __builtin_amdgcn_raw_buffer_load_b16(rm, threadIdx.x * 2u, 0, 0);
        else
            v.bits = __builtin_amdgcn_raw_buffer_load_b8(rm, threadIdx.x, 0, 0);
        const __amdgpu_buffer_rsrc_t rt = make_rsrc(in.tri + q, n * 4u);
        const __amdgpu_buffer_rsrc_t rn = make_rsrc(PACKED ? in.tri : in.node + q, n * 4u);
#pragma unroll
        for (uint32_t k = 0; k < PPT; ++k) {
            const uint32_t o = (threadIdx.x * PPT + k) * 4u;
            v.tri[k] = __builtin_amdgcn_raw_buffer_load_b32(rt, o, 0, 0);
            if constexpr (!PACKED) v.par[k] = __builtin_amdgcn_raw_buffer_load_b32(rn, o, 0, 0);
        }
        v.off = S.off[(t < ntiles ? t : 0u) + zero];
    };
    // nodes of the level below the one written, by 32-bit byte offsets (node
    // indices stay below 2^28)
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(na, ((uint64_t)off2 + n2) * 16u);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(nb, ((uint64_t)off2 + n2) * 16u);
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(ns, ((uint64_t)off2 + n2) * 4u);
    uint32_t wlo = 0u, wlen = 0u;           // nodes whose children are in LDS (block-uniform)
    uint32_t wend = 0u;                     // children of the copy's frame from the copy's first child on
    uint32_t wfull = 0u;                    // nodes of the copy with NF children each
    uint64_t tests64 = 0;                   // this wave's
    uint32_t parity = 0u;
    uint64_t prev_tile = 0;                 // first next-level tile of s_next
    if (TEST && threadIdx.x < NF + 2) s_next[threadIdx.x] = 0u;
    uint32_t tile = blockIdx.x * ch;
    tile_in next;
    if (tile < ntiles) load_tile(tile, next);
    for (; tile < ntiles; tile = next_of(tile), parity ^= 1u) {
        const tile_in cur = next;
        load_tile(next_of(tile), next);
        const uint32_t q0 = threadIdx.x * PPT;
        const uint32_t nq = (uint32_t)min(nin - (uint64_t)tile * TILE, (uint64_t)TILE);
        const uint32_t bits_in = PPT == 2 && q0 + 1 >= nq ? (q0 < nq ? cur.bits & 0xFFu : 0u) : cur.bits;
        uint32_t mk_[PPT], tri[PPT], first[PPT];
#pragma unroll
        for (uint32_t k = 0; k < PPT; ++k) {
            mk_[k] = PPT == 2 ? (bits_in >> (8 * k)) & 0xFFu : bits_in;
            uint32_t par;
            if constexpr (PACKED) {
                tri[k] = in.tri_base + (cur.tri[k] & ((1u << CRSH_PACKED_TRI_BITS) - 1u));
                par = cur.tri[k] >> CRSH_PACKED_TRI_BITS;
            } else {
                tri[k] = cur.tri[k];
                par = cur.par[k];
            }
            first[k] = par * F;
            if constexpr (BATCH) first[k] = mk_[k] && par < np ? bd.node_first[offp + par] : 0u;
        }
        const uint32_t mine = (uint32_t)__popc(bits_in);
        const uint32_t incl = wave_scan_dpp(mine);
        if (l == WAVE - 1) s_wave[parity][w] = incl;
        __syncthreads();
        // every wave is past the previous tile: its next-level sums go out
        if (TEST && threadIdx.x < NF + 2) {
            const uint32_t c = s_next[threadIdx.x];
            if (c) atomicAdd(&S.cnt[prev_tile + threadIdx.x], c);
            s_next[threadIdx.x] = 0u;
        }
        const uint64_t base = (uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(cur.off >> 32)) << 32 |
                              __builtin_amdgcn_readfirstlane((uint32_t)cur.off);
        prev_tile = base / TILE;
        // survivors of the waves before, and of the tile
        static_assert(NW == 8, "eight sums in the first lanes");
        uint32_t ws = l < NW ? s_wave[parity][l] : 0u;
        ws += dpp_from<0x111, 0xF>(0u, ws);
        ws += dpp_from<0x112, 0xF>(0u, ws);
        ws += dpp_from<0x114, 0xF>(0u, ws);
        const uint32_t n_out = __builtin_amdgcn_readlane(ws, NW - 1);
        uint32_t ex = incl - mine + (w ? __builtin_amdgcn_readlane(ws, w ? w - 1 : 0u) : 0u);
#pragma unroll
        for (uint32_t k = 0; k < PPT; ++k) {
            if (!mk_[k]) continue;
            const uint32_t p = threadIdx.x * PPT + k;
            s_par[p] = make_uint2(tri[k], first[k]);
#pragma unroll
            for (uint32_t c = 0; c < NF; ++c)
                if ((mk_[k] >> c) & 1u) s_item[ex++] = (uint16_t)(16u * p + c);
        }
        __syncthreads();
        if (n_out == 0u) continue;
        if constexpr (TEST && STAGED) {
            const uint32_t it = s_item[0];
            const uint32_t node = __builtin_amdgcn_readfirstlane(s_par[it >> 4].y + (it & 15u));
            if (node - wlo >= wlen) {
                // the frame's nodes on both levels, and its levels
                uint32_t pb = 0u, pc = n1, cb = 0u, cc = n2, levels = nl;
                if constexpr (BATCH) {
                    const uint32_t f = frame_of_node(bd, (uint32_t)parent_level - 2, node);
                    pb = bd.fm[f].level_base[parent_level - 2];
                    pc = bd.fm[f].level_cnt[parent_level - 2];
                    cb = bd.fm[f].level_base[parent_level - 3];
                    cc = bd.fm[f].level_cnt[parent_level - 3];
                    levels = bd.fm[f].n_levels;
                }
                uint32_t run = 1;               // a top-level node's descendants on the level written
                for (uint32_t k = 0; k + parent_level - 1 < levels && run <= WP; ++k) run *= F;
                wlen = wfull = 0u;
                if (run <= WP && node >= pb && node - pb < pc) {
                    wlo = pb + (node - pb) / run * run;
                    wlen = min(WP / run * run, pb + pc - wlo);
                    const uint32_t c0 = (wlo - pb) * F;
                    wend = cc - c0;
                    wfull = F == NF ? min(wlen, wend / NF) : 0u;
                    for (uint32_t r = 0; r < F; ++r)
                        for (uint32_t i = threadIdx.x; i < wlen; i += STEP_THREADS) {
                            const uint32_t c = i * F + r;
                            if (c >= wend) continue;
                            const uint32_t g = off2 + cb + c0 + c;
                            s_wa[r * WP + i] = na[g];
                            s_wb[r * WP + i] = nb[g];
                            s_ws[r * WP + i] = ns[g];
                        }
                    __syncthreads();
                }
            }
        }
        // what fits the storage; stores past it are dropped by their range
        const uint32_t n_put = base < out.cap ? (uint32_t)min(out.cap - base, (uint64_t)n_out) : 0u;
        const __amdgpu_buffer_rsrc_t ot = make_rsrc(out.tri + base, n_put * 4u);
        const __amdgpu_buffer_rsrc_t on = make_rsrc(PACKED ? out.tri : out.node + base, n_put * 4u);
        const __amdgpu_buffer_rsrc_t om = make_rsrc(mask_out + base, n_put * (uint32_t)sizeof(mask_t));
        // a written pair: triangle, node and (TEST) sphere; the next 64 are
        // requested before these are tested
        struct pair_in {
            uint32_t tri, node;
            float4 sp;
        };
        auto load_pair = [&](uint32_t i) {
            const uint32_t it = s_item[i < n_put ? i : 0u];
            const uint2 pr = s_par[it >> 4];
            pair_in v;
            v.tri = pr.x;
            v.node = pr.y + (it & 15u);
            if constexpr (TEST) v.sp = tsph[pr.x < m ? pr.x : 0u];
            return v;
        };
        pair_in pn;
        if (w * WAVE < n_put) pn = load_pair(w * WAVE + l);
        for (uint32_t i0 = w * WAVE; i0 < n_put; i0 += STEP_THREADS) {
            const uint32_t i = i0 + l;
            const pair_in cp = pn;
            const uint32_t node = cp.node;
            pn = load_pair(i + STEP_THREADS);
            if constexpr (PACKED) {
                __builtin_amdgcn_raw_buffer_store_b32(node << CRSH_PACKED_TRI_BITS | (cp.tri - out.tri_base), ot, i * 4u, 0, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b32(cp.tri, ot, i * 4u, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b32(node, on, i * 4u, 0, 0);
            }
            if constexpr (TEST) {
                const float4 sp = cp.sp;
                // first child and number of children of this lane's pair
                auto children = [&](uint32_t &c, uint32_t &k) {
                    c = node * F;
                    k = c < n2 ? min(F, n2 - c) : 0u;
                    if constexpr (BATCH) {
                        c = node < n1 ? bd.node_first[off1 + node] : 0u;
                        k = node < n1 ? bd.node_info[off1 + node] & INFO_COUNT_MASK : 0u;
                        k = c < n2 ? min(k, n2 - c) : 0u;
                    }
                };
                // the pair's pass bits, and the survivors of the lanes in the
                // first of the (at most two) next-level tiles they lie in
                const uint64_t p0 = base + i0;
                const uint32_t left = TILE - (uint32_t)(p0 % TILE);
                uint32_t bits = 0u, ca = 0u, cb = 0u;
                if constexpr (STAGED) {
                    const f3 pc = mk(sp.x, sp.y, sp.z);
                    const uint64_t live = n_put - i0 >= WAVE ? ~0ull : (1ull << (n_put - i0)) - 1ull;
                    const uint32_t pl = node - wlo;
                    uint64_t pass[NF];
                    // every pair's children in the copy, all F = NF of them: no
                    // looking further (a lane past the end repeats the first pair)
                    if (ballot(pl >= wfull) == 0) {
#pragma unroll
                        for (uint32_t r = 0; r < NF; ++r)
                            pass[r] = packed_meets_mask(s_wa[r * WP + pl], s_wb[r * WP + pl], s_ws[r * WP + pl], pc, sp.w) & live;
                        tests64 += (uint64_t)__popcll(live) * NF;
                    } else {
                        const bool inw = pl < wlen;
                        const uint32_t ps = inw ? pl : 0u;
                        uint32_t n = inw && i < n_put ? min(F, wend - pl * F) : 0u;
#pragma unroll
                        for (uint32_t r = 0; r < NF; ++r)
                            pass[r] = packed_meets_mask(s_wa[r * WP + ps], s_wb[r * WP + ps], s_ws[r * WP + ps], pc, sp.w) &
                                      ballot(r < n);
                        // pairs outside the copy: children from the node arrays
                        if (ballot(!inw && i < n_put) != 0) {
                            uint32_t c, k;
                            children(c, k);
                            k = !inw && i < n_put ? k : 0u;
                            n += k;
#pragma unroll
                            for (uint32_t r = 0; r < NF; ++r) {
                                const uint32_t g = off2 + (r < k ? c + r : 0u);
                                pass[r] |= packed_meets_mask(na[g], nb[g], ns[g], pc, sp.w) & ballot(r < k);
                            }
                        }
#pragma unroll
                        for (uint32_t r = 0; r < NF; ++r) tests64 += (uint64_t)__popcll(ballot(r < n));
                    }
                    const uint64_t in_first = left >= WAVE ? ~0ull : (1ull << left) - 1ull;
#pragma unroll
                    for (int r = NF - 1; r >= 0; --r) {
                        bits = bits + bits + (__builtin_amdgcn_inverse_ballot_w64(pass[r]) ? 1u : 0u);
                        ca += (uint32_t)__popcll(pass[r] & in_first);
                        cb += (uint32_t)__popcll(pass[r] & ~in_first);
                    }
                } else {
                    // lanes in groups of NF: in turn r a group tests the pair of
                    // its lane r, one child a lane
                    const uint32_t j = l % NF;
                    const int grp = (int)((l - j) * 4u);    // byte address of the group's first lane
                    auto turn = [&](uint32_t v, uint32_t r) {
                        return (uint32_t)__builtin_amdgcn_ds_bpermute(grp + (int)(4u * r), (int)v);
                    };
                    auto turnf = [&](float v, uint32_t r) { return __uint_as_float(turn(__float_as_uint(v), r)); };
                    uint32_t c, k;
                    children(c, k);
                    k = i < n_put ? k : 0u;
                    constexpr uint32_t K = 2;               // turns whose nodes are read together
#pragma unroll
                    for (uint32_t r0 = 0; r0 < NF; r0 += K) {
                        float4 A[K], Bv[K];
                        float Sg[K];
                        uint64_t ok[K];
#pragma unroll
                        for (uint32_t t = 0; t < K; ++t) {
                            const uint32_t first = turn(c, r0 + t);
                            const bool has = j < turn(k, r0 + t);
                            const uint32_t g = off2 + (has ? first + j : 0u);
                            ok[t] = ballot(has);
                            A[t] = buf_load4(ra, g * 16u);
                            Bv[t] = buf_load4(rb, g * 16u);
                            Sg[t] = buf_load1(rs, g * 4u);
                        }
#pragma unroll
                        for (uint32_t t = 0; t < K; ++t) {
                            const uint32_t r = r0 + t;
                            const uint64_t m = packed_meets_mask(A[t], Bv[t], Sg[t], mk(turnf(sp.x, r), turnf(sp.y, r),
                                                                 turnf(sp.z, r)), turnf(sp.w, r)) & ok[t];
                            tests64 += (uint64_t)__popcll(ok[t]);
                            ca += (uint32_t)__popcll(m);
                            bits = j == r ? (uint32_t)(m >> (l - j)) & ((1u << NF) - 1u) : bits;
                        }
                    }
                    if (left < WAVE) {
                        cb = wave_reduce(l < left ? 0u : (uint32_t)__popc(bits), 0u,
                                         [](uint32_t a, uint32_t b) { return a + b; });
                        ca -= cb;
                    }
                }
                if constexpr (sizeof(mask_t) == 1)
                    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)bits, om, i, 0, 0);
                else
                    __builtin_amdgcn_raw_buffer_store_b16((uint16_t)bits, om, i * 2u, 0, 0);
                const uint32_t k = (uint32_t)(p0 / TILE - prev_tile);
                if (l == 0 && ca) atomicAdd(&s_next[k], ca);
                if (l == 0 && cb) atomicAdd(&s_next[k + 1], cb);
            }
        }
    }
    if constexpr (TEST) {
        __syncthreads();
        if (threadIdx.x < NF + 2) {
            const uint32_t c = s_next[threadIdx.x];
            if (c) atomicAdd(&S.cnt[prev_tile + threadIdx.x], c);
        }
        __shared__ uint64_t s_tests[NW];
        if (l == 0) s_tests[w] = tests64;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint64_t sum = 0;
            for (uint32_t k = 0; k < NW; ++k) sum += s_tests[k];
            S.part[blockIdx.x] += sum;
        }
    }
}

// ------------------------------------------------------------------ scan
// Exclusive scan of the item counts into 64-bit offsets; the total becomes
// the pair count of the output level.  Tiles take their index from an atomic
// counter in launch order, so every tile waited on in the look-back has
// started and publishes its sum without waiting: the look-back always ends.
// There are few tiles (SCAN_TILE items each); a grid for every tile that the
// storage could hold would be thousands of blocks with nothing to do.
// A batch's top-level pass (batch_top = its level, 1-based) scans bd_top[0]
// items and appends after the bd_top[1] pairs already on that level.
// Level scans clear the counts they read (the next step adds into them), and
// one more block adds the workgroups' sums of the launch before to meta:
// three counts of the top-level count, or node tests.  A chain of latencies
// (ticket, counts, look-back) bounds it: 16 bytes of counts a thread.
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_items(int32_t parent_level, uint32_t n_mesh, uint32_t tile_pairs,
                                                             pair_levels P, trav_scratch S, crsh_meta *meta,
                                                             uint32_t batch_top, const uint64_t *bd_top,
                                                             uint32_t blocks)
{
    __shared__ uint32_t s_tile;
    __shared__ uint64_t s_excl;
    __shared__ uint64_t s_scan[3][SCAN_THREADS / WAVE];
    const uint32_t nl = meta->n_levels;
    if (nl == 0) return;
    if (batch_top > nl) return;
    const bool top = parent_level == 0;
    uint32_t parts;
    const uint64_t n = batch_top ? bd_top[0] : level_items(meta, parent_level, n_mesh, P, tile_pairs, S.top_cap, S.top_many, parts);
    const uint64_t base = batch_top ? bd_top[1] : 0u;
    const uint32_t out_level = batch_top ? batch_top - 1 : (top ? nl - 1 : (uint32_t)parent_level - 2);
    const uint64_t ntiles = (n + SCAN_TILE - 1) / SCAN_TILE;
    // the last block: the launch before's workgroup sums (three for the
    // top-level count)
    if (blockIdx.x == gridDim.x - 1) {
        if (n == 0) return;                 // the sums are of a level further down
        uint64_t c[3] = {0, 0, 0};
        for (uint32_t i = threadIdx.x; i < blocks; i += SCAN_THREADS) {
            if (top) {
                for (uint32_t k = 0; k < 3; ++k) c[k] += S.top_part[3 * i + k];
            } else {
                c[0] += S.part[i];
                S.part[i] = 0u;
            }
        }
        const uint32_t kinds = top ? 3u : 1u;
        for (uint32_t k = 0; k < kinds; ++k) {
            c[k] = wave_sum(c[k]);
            if (lane_id() == 0) s_scan[k][threadIdx.x / WAVE] = c[k];
        }
        __syncthreads();
        if (threadIdx.x < kinds) {
            uint64_t t = 0;
            for (uint32_t w = 0; w < SCAN_THREADS / WAVE; ++w) t += s_scan[threadIdx.x][w];
            uint64_t *const dst = threadIdx.x == 0 ? &meta->tests[out_level]
                                : threadIdx.x == 1 ? &meta->mesh_hits : &meta->mesh_tests;
            *dst += t;
        }
        return;
    }
    if (blockIdx.x >= ntiles) return;       // only ntiles blocks take a tile
    uint32_t *const cnt = top ? S.cnt_top : S.cnt;
    for (;;) {
        uint32_t tile = 0;
        if (ntiles > 1) {
            if (threadIdx.x == 0) s_tile = atomicAdd(S.scan_ctr, 1u);
            __syncthreads();
            tile = s_tile;
            if (tile >= ntiles) return;
        }
        const uint64_t first = (uint64_t)tile * SCAN_TILE + (uint64_t)threadIdx.x * SCAN_ITEMS;
        static_assert(SCAN_ITEMS == 4, "16 bytes of counts per thread");
        uint32_t v[SCAN_ITEMS] = {0u, 0u, 0u, 0u};
        const bool whole = first + SCAN_ITEMS <= n;
        if (whole) {
            const uint4 x = *(const uint4 *)(cnt + first);
            v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
        } else {
#pragma unroll
            for (uint32_t k = 0; k < SCAN_ITEMS; ++k)
                if (first + k < n) v[k] = cnt[first + k];
        }
        const uint64_t sum = ((uint64_t)v[0] + v[1]) + ((uint64_t)v[2] + v[3]);
        uint64_t total;
        const uint64_t ex = block_excl_scan<uint64_t, SCAN_THREADS / WAVE>(sum, s_scan[0], total);
        if (ntiles > 1) {
            if (threadIdx.x < WAVE) {
                const uint64_t e = lookback_wave(S.scan_flags, tile, total);
                if (threadIdx.x == 0) s_excl = e;
            }
            __syncthreads();
        }
        uint64_t run = base + ex + (ntiles > 1 ? s_excl : 0u);
        if (tile == ntiles - 1 && threadIdx.x == SCAN_THREADS - 1) {
            const uint64_t end = run + sum;
            meta->pairs[out_level] = end;
            atomicAdd((unsigned long long *)&meta->hits[out_level], (unsigned long long)(end - base));
            if (end > P.p[out_level].cap) atomicOr(&meta->status, CRSH_OVERFLOW_PAIRS);
        }
        if (whole) {
            const uint64_t o1 = run + v[0], o2 = o1 + v[1], o3 = o2 + v[2];
            typedef uint64_t v2 __attribute__((ext_vector_type(2)));
            *(v2 *)(S.off + first) = v2{run, o1};
            *(v2 *)(S.off + first + 2) = v2{o2, o3};
            if (!top) *(uint4 *)(cnt + first) = make_uint4(0u, 0u, 0u, 0u);
        } else {
#pragma unroll
            for (uint32_t k = 0; k < SCAN_ITEMS; ++k) {
                if (first + k < n) {
                    S.off[first + k] = run;
                    if (!top) cnt[first + k] = 0u;
                }
                run += v[k];
            }
        }
        if (ntiles == 1) return;
    }
}

// Batch, before the top-level pass of level L: item ranges of the frames
// whose top is L (one thread per frame), their total, and the pairs already
// on that level (the append base).  Too many items: flagged, pass skipped.
__global__ __launch_bounds__(256) void k_batch_top_plan(batch_dev bd, crsh_meta *meta, uint32_t L, uint32_t many)
{
    __shared__ uint64_t scratch[256 / WAVE];
    const uint32_t f = threadIdx.x;
    const bool live = f < bd.n_frames;
    uint64_t items = 0;
    if (live && bd.fm[f].n_levels == L && L >= 1)
        items = (uint64_t)bd.fm[f].level_cnt[L - 1] * bd.frames[f].mesh_count;
    uint64_t total;
    const uint64_t ex = block_excl_scan<uint64_t, 256 / WAVE>(items, scratch, total);
    if (live) bd.fm[f].item_base = ex;
    if (f == 0) {
        if (total > bd.top_cap) {
            atomicOr(&meta->status, CRSH_OVERFLOW_ITEMS);
            total = 0;
        }
        const uint32_t parts = top_parts(total, bd.top_cap, many);
        bd.top[0] = total * parts;
        bd.top[2] = parts;
        bd.top[1] = L >= 1 ? meta->pairs[L - 1] : 0u;
    }
}

}  // namespace crsh

using namespace crsh;

namespace crsh {

void trav_prep_launch(const crsh_scene *scene, uint32_t tri_begin, uint32_t tri_end, float4 *tsph,
                      const crsh_nodes *nodes, crsh_meta *meta, float4 *na, float4 *nb, float *ns,
                      const trav_scratch &S, uint64_t n_cnt, uint32_t levels, hipStream_t stream)
{
    const node_arrays nd{nodes->cx, nodes->cy, nodes->cz, nodes->r, nodes->ax, nodes->ay, nodes->az,
                         nodes->c, nodes->tan, nodes->sec};
    tri_verts V;
    for (int k = 0; k < 9; ++k) V.v[k] = scene->v[k];
    uint64_t items = std::max(std::max<uint64_t>(nodes->capacity, n_cnt), (uint64_t)(tri_end - tri_begin));
    items = std::max<uint64_t>(items, TRAV_PARTS);
    const uint32_t g = (uint32_t)std::min<uint64_t>((items + 255) / 256, 4096);
    k_trav_prep<<<g, 256, 0, stream>>>(V, tri_begin, tri_end, tsph, nd, meta, na, nb, ns, S, n_cnt, levels);
}

void level_count_launch(int32_t parent_level, int32_t merge, const float4 *na, const float4 *nb, const float *ns,
                        const float4 *tsph, uint32_t m, const pair_levels &P, const trav_scratch &S, crsh_meta *meta,
                        const batch_dev *bd, uint64_t tiles_cap, uint32_t top_levels, hipStream_t stream)
{
    const batch_dev b = bd ? *bd : batch_dev{};
    const uint32_t Fu = (uint32_t)merge;
    const int L = parent_level;
    int nf = 2;
    while (nf < merge) nf *= 2;
    // descendants of a top-level node on the child level, for a hierarchy
    // of at most top_levels levels: the staged kernel if they fit the window
    uint64_t run = 1;
    for (int e = 0; e < (int)top_levels - L + 1 && run <= COUNT_WINDOW; ++e) run *= Fu;
    const bool st = run <= COUNT_WINDOW;
    prof_scope ps("k_level", stream);
    // a persistent grid of one round of resident blocks (at most one block
    // per step of COUNT_TPS tiles)
#define CRSH_COUNT_ONE(NF, BT, ST)                                                                           \
    {                                                                                                        \
        const uint32_t rb = resident_blocks((const void *)k_level_count_lanes<NF, BT, ST>, COUNT_THREADS);                 \
        const uint64_t want = std::max<uint64_t>((tiles_cap + COUNT_TPS - 1) / COUNT_TPS, 1);                \
        const uint32_t gl = (uint32_t)std::min<uint64_t>(want, rb ? rb : 2048);                              \
        k_level_count_lanes<NF, BT, ST><<<gl, COUNT_THREADS, 0, stream>>>(L, Fu, na, nb, ns, tsph, m, P, S,  \
                                                                        meta, b);                           \
    }
#define CRSH_COUNT_ST(NF, BT)                                                                                \
    if (st)                                                                                                  \
        CRSH_COUNT_ONE(NF, BT, true)                                                                         \
    else                                                                                                     \
        CRSH_COUNT_ONE(NF, BT, false)
#define CRSH_COUNT_NF(BT)                                                                                    \
    switch (nf) {                                                                                            \
    case 2: CRSH_COUNT_ST(2, BT) break;                                                                      \
    case 4: CRSH_COUNT_ST(4, BT) break;                                                                      \
    case 8: CRSH_COUNT_ST(8, BT) break;                                                                      \
    default: CRSH_COUNT_ST(16, BT) break;                                                                    \
    }
    if (bd) {
        CRSH_COUNT_NF(true)
    } else {
        CRSH_COUNT_NF(false)
    }
#undef CRSH_COUNT_NF
#undef CRSH_COUNT_ST
#undef CRSH_COUNT_ONE
}

// lowest: the lowest level produced (1, or 2 when crsh_leaf_hit forms the
// level-1 pairs itself); a top-level pass always writes its own level.
// P: the pair storage of `levels` consecutive levels (largest capacity
// max_pairs), unpacked or packed.
static crsh_status traverse_run(const crsh_nodes *nodes, const crsh_scene *scene, uint32_t tri_begin,
                                uint32_t tri_end, int32_t bundle, int32_t merge, const pair_levels &P, int levels,
                                uint64_t max_pairs, crsh_meta *meta, void *ws, size_t ws_bytes, const batch_dev *bd,
                                int32_t batch_levels, uint64_t batch_top_items, int32_t lowest, hipStream_t stream)
{
    if (!nodes || !scene || !meta || !ws) {
        set_error("crsh_traverse: NULL argument");
        return CRSH_ERR_INVALID;
    }
    if (bundle < 1 || bundle > CRSH_MAX_BUNDLE || merge < 2 || merge > CRSH_MAX_MERGE) {
        set_error("crsh_traverse: bad bundle or merge factor");
        return CRSH_ERR_INVALID;
    }
    for (int k = 0; k < 9; ++k)
        if (!scene->v[k] && scene->m) {
            set_error("crsh_traverse: missing vertex array");
            return CRSH_ERR_INVALID;
        }
    if (scene->n_mesh == 0 || !scene->mesh_first || !scene->mesh_count || !scene->msph) {
        set_error("crsh_traverse: scene has no meshes");
        return CRSH_ERR_INVALID;
    }
    if (tri_end > scene->m || tri_begin > tri_end) {
        set_error("crsh_traverse: triangle batch [%u, %u) outside [0, %u)", tri_begin, tri_end, scene->m);
        return CRSH_ERR_INVALID;
    }
    if (lowest < 1 || lowest > 2) {
        set_error("crsh_traverse: lowest level must be 1 or 2");
        return CRSH_ERR_INVALID;
    }
    if (levels == 0) {
        set_error("crsh_traverse: no pair storage");
        return CRSH_ERR_INVALID;
    }
    if (bd && levels < batch_levels) {
        set_error("crsh_batch: pair storage for %d levels, %d needed", levels, batch_levels);
        return CRSH_ERR_INVALID;
    }
    const bool packed = P.p[0].packed != 0;
    if (packed && bd) {
        set_error("crsh_batch: packed pairs are not supported in the batched form");
        return CRSH_ERR_INVALID;
    }
    const uint64_t top_items = bd ? batch_top_items : (uint64_t)nodes->capacity * scene->n_mesh;
    size_t need = trav_ws_bytes(scene->m, nodes->capacity, top_items, max_pairs);
    if (ws_bytes < need) {
        set_error("crsh_traverse: workspace too small (%zu < %zu)", ws_bytes, need);
        return CRSH_ERR_INVALID;
    }
    const uint64_t tiles = max_pairs / STEP_THREADS + 2;       // at least step_tile pairs each
    const uint64_t items = std::max(top_items, tiles) + 1;
    char *w = (char *)ws;
    float4 *tsph = (float4 *)w;
    w += align256((size_t)scene->m * 16);
    float4 *na = (float4 *)w;
    w += align256((size_t)nodes->capacity * 16);
    float4 *nb = (float4 *)w;
    w += align256((size_t)nodes->capacity * 16);
    float *ns = (float *)w;
    w += align256((size_t)nodes->capacity * 4);
    trav_scratch S{};
    S.top_cap = top_items;
    S.top_many = top_many(scene->m, scene->n_mesh);
    S.cnt_top = (uint32_t *)w;
    w += align256(top_items * 4 + 4);
    S.cnt = (uint32_t *)w;
    w += align256(tiles * 4);
    S.off = (uint64_t *)w;
    w += align256(items * 8);
    S.mask[0] = w;
    w += align256(max_pairs * 2 + 2);
    S.mask[1] = w;
    w += align256(max_pairs * 2 + 2);
    S.scan_flags = (uint64_t *)w;
    S.n_flags = (uint32_t)(items / SCAN_TILE + 2);
    w += align256((items / SCAN_TILE + 2) * 8);
    S.scan_ctr = (uint32_t *)w;
    w += align256(4);
    S.part = (uint64_t *)w;
    S.top_part = S.part + TRAV_PARTS;

    int nf = 2;
    while (nf < merge) nf *= 2;
    const uint32_t tile_pairs = step_tile(nf);
    const batch_dev b = bd ? *bd : batch_dev{};
    trav_prep_launch(scene, tri_begin, tri_end, tsph, nodes, meta, na, nb, ns, S, max_pairs / tile_pairs + 1,
                     (uint32_t)levels, stream);
    const uint32_t scan_grid = (uint32_t)std::min<uint64_t>((items + SCAN_TILE - 1) / SCAN_TILE, SCAN_GRID);
    // one wave per top-level item, for the items that a hierarchy with as many
    // levels as there is storage for has (more items loop)
    uint64_t top_est = top_items;
    if (!bd) {
        uint64_t n = nodes->capacity;
        for (int k = 1; k < levels && n > 1; ++k) n = (n + merge - 1) / merge;
        top_est = n * scene->n_mesh;
    }
    const uint32_t top_grid = (uint32_t)std::min<uint64_t>(std::max<uint64_t>((top_est + 3) / 4, 256), 2048);
    static_assert(TRAV_PARTS >= 2048, "a sum per workgroup of the top-level passes");
    const uint32_t Fu = (uint32_t)merge;
#define CRSH_NF(DO)              \
    switch (nf) {                \
    case 2: DO(2); break;        \
    case 4: DO(4); break;        \
    case 8: DO(8); break;        \
    default: DO(16); break;      \
    }

    // top-level pass: plain (L = 0, the one top level) or a batch level L
    auto top_pass_launch = [&](uint32_t L) {
        if (bd) k_batch_top_plan<<<1, 256, 0, stream>>>(b, meta, L, S.top_many);
        {
            prof_scope ps("k_top_count", stream);
            if (bd)
                k_top_count<true><<<top_grid, 256, 0, stream>>>(na, nb, ns, tsph, scene->mesh_first,
                                                                scene->mesh_count, scene->msph, scene->n_mesh,
                                                                tri_begin, tri_end, P, S, meta, b, L);
            else
                k_top_count<false><<<top_grid, 256, 0, stream>>>(na, nb, ns, tsph, scene->mesh_first,
                                                                 scene->mesh_count, scene->msph, scene->n_mesh,
                                                                 tri_begin, tri_end, P, S, meta, b, L);
        }
        k_scan_items<<<scan_grid + 1, SCAN_THREADS, 0, stream>>>(0, scene->n_mesh, tile_pairs, P, S, meta, L, b.top,
                                                             top_grid);
        prof_scope ps("k_top_emit", stream);
#define CRSH_TOP(NF, BT, PK)                                                                                      \
    k_top_emit<NF, BT, PK><<<top_grid, 256, 0, stream>>>(na, nb, ns, tsph, scene->mesh_first, scene->mesh_count,  \
                                                         scene->msph, scene->n_mesh, tri_begin, tri_end, Fu,      \
                                                         (uint32_t)lowest, P, S, meta, b, L)
#define CRSH_TOP_BATCH(NF) CRSH_TOP(NF, true, false)
#define CRSH_TOP_PACKED(NF) CRSH_TOP(NF, false, true)
#define CRSH_TOP_PLAIN(NF) CRSH_TOP(NF, false, false)
        if (bd) {
            CRSH_NF(CRSH_TOP_BATCH)
        } else if (packed) {
            CRSH_NF(CRSH_TOP_PACKED)
        } else {
            CRSH_NF(CRSH_TOP_PLAIN)
        }
#undef CRSH_TOP_BATCH
#undef CRSH_TOP_PACKED
#undef CRSH_TOP_PLAIN
#undef CRSH_TOP
    };
    // one level step: pairs of level L (1-based parent) -> level L - 1, tested
    // against level L - 2 if another step follows
    const uint32_t top_levels = (uint32_t)(bd ? batch_levels : levels);
    uint32_t parts = top_grid;               // workgroups that may have left a sum of node tests
    auto level_step_launch = [&](int L) {
        k_scan_items<<<scan_grid + 1, SCAN_THREADS, 0, stream>>>(L, scene->n_mesh, tile_pairs, P, S, meta, 0, nullptr,
                                                             parts);
        const uint64_t want = std::max<uint64_t>((P.p[L - 1].cap + tile_pairs - 1) / tile_pairs, 1);
        const bool test = L - 1 > lowest;
        // a top-level node's descendants on the level written, in a hierarchy
        // of at most top_levels levels: the copying kernel if their children
        // fit the copy
        uint64_t run = (uint64_t)nf;
        for (int k = L - 1; k < (int)top_levels && run <= COUNT_WINDOW; ++k) run *= Fu;
        const bool st = run <= COUNT_WINDOW;
        prof_scope ps("k_level", stream), pe("k_level_emit", stream);
#define CRSH_STEP(NF, BT, PK, TE, ST)                                                                             \
    {                                                                                                             \
        const uint32_t rb = resident_blocks((const void *)k_level_step<NF, BT, PK, TE, ST>, STEP_THREADS);                      \
        const uint32_t g = (uint32_t)std::min<uint64_t>(want, std::min(rb ? rb : 512u, TRAV_PARTS));              \
        parts = std::max(parts, g);                                                                               \
        k_level_step<NF, BT, PK, TE, ST><<<g, STEP_THREADS, 0, stream>>>(L, Fu, na, nb, ns, tsph, scene->m, P, S, \
                                                                         meta, b);                               \
    }
#define CRSH_STEP_T(NF, BT, PK)                  \
    if (!test)                                   \
        CRSH_STEP(NF, BT, PK, false, false)      \
    else if (st)                                 \
        CRSH_STEP(NF, BT, PK, true, true)        \
    else                                         \
        CRSH_STEP(NF, BT, PK, true, false)
#define CRSH_STEP_BATCH(NF) CRSH_STEP_T(NF, true, false)
#define CRSH_STEP_PACKED(NF) CRSH_STEP_T(NF, false, true)
#define CRSH_STEP_PLAIN(NF) CRSH_STEP_T(NF, false, false)
        if (bd) {
            CRSH_NF(CRSH_STEP_BATCH)
        } else if (packed) {
            CRSH_NF(CRSH_STEP_PACKED)
        } else {
            CRSH_NF(CRSH_STEP_PLAIN)
        }
#undef CRSH_STEP_BATCH
#undef CRSH_STEP_PACKED
#undef CRSH_STEP_PLAIN
#undef CRSH_STEP_T
#undef CRSH_STEP
    };
    if (bd) {
        for (int L = batch_levels; L >= 1; --L) {
            if (L < batch_levels && L >= lowest) level_step_launch(L + 1);
            top_pass_launch((uint32_t)L);
        }
    } else {
        top_pass_launch(0);
        for (int L = levels; L >= lowest + 1; --L) level_step_launch(L);
    }
#undef CRSH_NF
    return hip_check(hipGetLastError(), "crsh_traverse launch");
}

crsh_status traverse_launch(const crsh_nodes *nodes, const crsh_scene *scene, uint32_t tri_begin, uint32_t tri_end,
                            int32_t bundle, int32_t merge, const crsh_pairs pairs[CRSH_MAX_LEVELS],
                            crsh_meta *meta, void *ws, size_t ws_bytes, const batch_dev *bd, int32_t batch_levels,
                            uint64_t batch_top_items, int32_t lowest, hipStream_t stream)
{
    if (!pairs) {
        set_error("crsh_traverse: NULL argument");
        return CRSH_ERR_INVALID;
    }
    // levels present in the pair table: consecutive entries with storage
    pair_levels P{};
    int levels = 0;
    uint64_t max_pairs = 0;
    while (levels < CRSH_MAX_LEVELS && pairs[levels].tri && pairs[levels].node) {
        P.p[levels].tri = pairs[levels].tri;
        P.p[levels].node = pairs[levels].node;
        P.p[levels].cap = pairs[levels].capacity;
        max_pairs = std::max(max_pairs, pairs[levels].capacity);
        ++levels;
    }
    return traverse_run(nodes, scene, tri_begin, tri_end, bundle, merge, P, levels, max_pairs, meta, ws, ws_bytes,
                        bd, batch_levels, batch_top_items, lowest, stream);
}

// packed pairs need every level's node ids below 2^(32 - CRSH_PACKED_TRI_BITS)
__global__ void k_packed_check(crsh_meta *meta)
{
    const uint32_t nl = min(meta->n_levels, (uint32_t)CRSH_MAX_LEVELS);
    for (uint32_t k = 0; k < nl; ++k)
        if (meta->level_cnt[k] > CRSH_PACKED_MAX_NODES) atomicOr(&meta->status, CRSH_OVERFLOW_PACKED);
}

}  // namespace crsh

extern "C" crsh_status crsh_traverse_packed(const crsh_nodes *nodes, const crsh_scene *scene, uint32_t tri_begin,
                                            uint32_t tri_end, int32_t bundle, int32_t merge,
                                            const crsh_packed_pairs pairs[CRSH_MAX_LEVELS], crsh_meta *meta,
                                            void *ws, size_t ws_bytes, hipStream_t stream)
{
    if (!pairs || !meta) {
        set_error("crsh_traverse_packed: NULL argument");
        return CRSH_ERR_INVALID;
    }
    if (tri_begin > tri_end || tri_end - tri_begin > CRSH_PACKED_MAX_TRIS) {
        set_error("crsh_traverse_packed: a triangle batch holds at most %u triangles (got [%u, %u))",
                  CRSH_PACKED_MAX_TRIS, tri_begin, tri_end);
        return CRSH_ERR_INVALID;
    }
    pair_levels P{};
    int levels = 0;
    uint64_t max_pairs = 0;
    while (levels < CRSH_MAX_LEVELS && pairs[levels].pair) {
        P.p[levels].tri = pairs[levels].pair;
        P.p[levels].node = nullptr;
        P.p[levels].cap = pairs[levels].capacity;
        P.p[levels].packed = 1;
        P.p[levels].tri_base = tri_begin;
        max_pairs = std::max(max_pairs, pairs[levels].capacity);
        ++levels;
    }
    crsh_status st = traverse_run(nodes, scene, tri_begin, tri_end, bundle, merge, P, levels, max_pairs, meta, ws,
                                  ws_bytes, nullptr, 0, 0, 1, stream);
    if (st != CRSH_OK) return st;
    k_packed_check<<<1, 1, 0, stream>>>(meta);
    return hip_check(hipGetLastError(), "crsh_traverse_packed launch");
}

extern "C" crsh_status crsh_traverse(const crsh_nodes *nodes, const crsh_scene *scene, uint32_t tri_begin,
                                     uint32_t tri_end, int32_t bundle, int32_t merge,
                                     const crsh_pairs pairs[CRSH_MAX_LEVELS], crsh_meta *meta, void *ws,
                                     size_t ws_bytes, hipStream_t stream)
{
    return traverse_launch(nodes, scene, tri_begin, tri_end, bundle, merge, pairs, meta, ws, ws_bytes, nullptr, 0,
                           0, 1, stream);
}

extern "C" crsh_status crsh_traverse_upper(const crsh_nodes *nodes, const crsh_scene *scene, uint32_t tri_begin,
                                           uint32_t tri_end, int32_t bundle, int32_t merge,
                                           const crsh_pairs pairs[CRSH_MAX_LEVELS], crsh_meta *meta, void *ws,
                                           size_t ws_bytes, hipStream_t stream)
{
    return traverse_launch(nodes, scene, tri_begin, tri_end, bundle, merge, pairs, meta, ws, ws_bytes, nullptr, 0,
                           0, 2, stream);
}
