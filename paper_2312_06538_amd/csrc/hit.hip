// Stage 5: final intersection tests and closest hit (Sec. 3.3.8).
//
// k_hit_pack   ray slots (below), and triangles repacked twice: 3 x float4
//              (v0, e1 = v1 - v0, e2 = v2 - v0; e1, e2 are the same single
//              roundings the test would make) for the test itself, and
//              3 x float4 of the filter (below) with its error bound.
// k_hit        persistent workgroups over the level-1 pairs: a chunk of pairs
//              is binned by leaf in LDS, each leaf's rays are tested against
//              its triangles with matrix instructions, and what that filter
//              cannot reject goes through the test as written (the fused form
//              reads level-2 pairs and the pass bits of their children).  A hit
//              lowers the ray's 64-bit (order-mapped t, triangle) key with an
//              atomic minimum: the closest hit, ties to the lower triangle id.
// k_hit_final  one thread per sorted ray: decode the key, recompute u, v with
//              the same test, write the result at the ray id.
// Ray slots: k_hit reads the rays of leaf l at slots l * B + j, j < B, of
// three packed arrays of 16 bytes a slot: (origin, tmax), (direction, its
// length) and, with the origin o taken from a point of the scene, (o x direction,
// |o| |direction|); the interval start t_min is the frame's.  In the plain form
// slot s is sorted ray s.  In the batched form a frame's rays are bundled B at a
// time from its own first ray, so only a frame's last leaf can hold fewer than B
// rays; its slots are padded (zeros, a length of -1) and the closest-hit keys are
// kept by slot, so the pair loop finds a ray with no per-leaf lookup.
// k_hit_final maps each sorted ray back to its slot through its frame's first
// leaf and first ray.
#include "batch.hpp"
#include "intersect.hpp"

namespace crsh {

// The filter.  The test accepts u = a / det in [0, 1] with
// a = (O - v0) . (D x e2) and det = e1 . (D x e2), i.e. |2 a - det| <= |det|.
// With o = O - C and w = v0 - C for a point C of the scene, and the ray's moment
// M = o x D, both are sums of products of one ray vector and one triangle vector,
//     2 a - det = M . (2 e2) - D . (2 e2 x w + e2 x e1),   det = D . (e2 x e1),
// so a leaf's rays against its triangles are a small matrix product.  A pair
// is rejected when |2 a - det| - |det| > T with
//     T = 2^-18 |e2| |D| (|o| + |w| + |e1|).
// Error bound (u = 2^-24, first order): the two forms above come out within
// u |e2||D| (21 |o| + 23 |w| + 10.5 |e1|), of which rounding o and w is 2 |o| and
// 2 |w|, and 6.5 u |e1||e2||D|; the test's own a and det within
// 7.5 u |e2||D| (|o| + |w|) and 6.5 u |e1||e2||D|; and 16 u |e1||e2||D| more keeps
// a / det 2^-21 away from 0 and 1, so that the rounded quotient falls on the same
// side: together at most u |e2||D| (36 |o| + 38 |w| + 46 |e1|), against T's 64 u.
// What T is next to |e2||D||e1| decides how much is rejected: at distances of 2^12
// edges a few tests in a hundred that fail are made in full, at 2^18 all.  So C
// keeps a scene far from the origin as cheap as one around it (512x512 reflections,
// a scene 60 across moved by 10^5: final tests 2.15 ms with C = 0 and T twice as
// large, 0.88 so, 0.73 around the origin).  Rays from far away stay dearer: shadow
// rays of a scene 100 across with its light at 10^5 0.43 ms (0.35 with a lane a test
// and no filter, 0.53 with T twice as large), at 10^6 2.1 (1.3, 2.5).  Where a length
// is above 2^40, or |D| below 2^-40, or one is a NaN, a product could overflow or
// underflow: such a triangle has zero vectors and a large T, such a ray a mark,
// and neither is ever rejected, which takes 1.7 times as long as a test did
// without the filter.  In these bounds no product of the filter or of the test's
// a and det exceeds 2^122, and T is at least 2^-18 2^-30 2^-40 (3 2^-30) > 2^-117
// (FLT_TINY), against the at most 2^-122 that products below the normal range
// lose in the nine terms of 2 a - det and det.
constexpr float FLT_REL = 0x1p-18f;
constexpr float FLT_TINY = 0x1p-30f;       // added to lengths: their squares may underflow
constexpr float FLT_LONG = 0x1p40f, FLT_SHORT = 0x1p-40f;
constexpr float FLT_KEEP = -2.0f;          // |O||D| of a ray that the filter may not reject

// C: by coordinate the middle one of three vertices of triangles a quarter, half
// and three quarters through the scene, so that few outliers do not matter.  Any C
// is right; in a batch of frames it is the same for all.
__device__ __forceinline__ f3 filter_centre(const tri_verts &V, uint32_t m)
{
    if (m == 0u) return mk(0.0f, 0.0f, 0.0f);
    const uint32_t a = m / 4, b = m / 2, d = m - 1u - m / 4;
    const f3 c = mk(__builtin_amdgcn_fmed3f(V.v[0][a], V.v[0][b], V.v[0][d]),
                    __builtin_amdgcn_fmed3f(V.v[1][a], V.v[1][b], V.v[1][d]),
                    __builtin_amdgcn_fmed3f(V.v[2][a], V.v[2][b], V.v[2][d]));
    const bool ok = fabsf(c.x) <= FLT_LONG && fabsf(c.y) <= FLT_LONG && fabsf(c.z) <= FLT_LONG;     // no NaN
    return ok ? c : mk(0.0f, 0.0f, 0.0f);
}

// Per triangle: (2 e2, E0), (-(2 e2 x w + e2 x e1), E1), (e2 x e1, 0) with
// T = E0 |o||D| + E1 |D|.  Entry m pads a leaf's last triangles: its T is
// negative for every ray (rejected).
__device__ __forceinline__ void put_tri(const tri_verts &V, uint32_t t, uint32_t m, f3 centre, const hit_tris_ws &out)
{
    float4 *const tri = out.tri + 3 * (size_t)t, *const ftri = out.ftri + 3 * (size_t)t;
    if (t == m) {
        ftri[0] = make_float4(0.0f, 0.0f, 0.0f, -1.0f);
        ftri[1] = make_float4(0.0f, 0.0f, 0.0f, 0x1p-60f);
        ftri[2] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        return;
    }
    const f3 a = mk(V.v[0][t], V.v[1][t], V.v[2][t]);
    const f3 e1 = mk(V.v[3][t], V.v[4][t], V.v[5][t]) - a;
    const f3 e2 = mk(V.v[6][t], V.v[7][t], V.v[8][t]) - a;
    tri[0] = make_float4(a.x, a.y, a.z, e1.x);
    tri[1] = make_float4(e1.y, e1.z, e2.x, e2.y);
    tri[2] = make_float4(e2.z, 0.0f, 0.0f, 0.0f);
    const f3 ac = a - centre;
    const float la = len(ac) + FLT_TINY, l1 = len(e1) + FLT_TINY, l2 = len(e2) + FLT_TINY;
    const bool ok = la <= FLT_LONG && l1 <= FLT_LONG && l2 <= FLT_LONG;
    const f3 z = mk(0.0f, 0.0f, 0.0f);
    const f3 n = ok ? cross(e2, e1) : z;
    const f3 w = ok ? cross(e2, ac) * 2.0f + n : z;
    const f3 e = ok ? e2 * 2.0f : z;
    ftri[0] = make_float4(e.x, e.y, e.z, ok ? FLT_REL * l2 : 0.0f);
    ftri[1] = make_float4(-w.x, -w.y, -w.z, ok ? FLT_REL * l2 * (la + l1) : 0x1p60f);
    ftri[2] = make_float4(n.x, n.y, n.z, 0.0f);
}

struct sorted_rays {
    const float *ox, *oy, *oz, *dx, *dy, *dz, *tmax;
};

// tmax word of a padded slot (a NaN); a NaN tmax of a real ray is stored as
// the default quiet NaN, which accepts no hit either
constexpr uint32_t PAD_SLOT = 0x7FC0DEADu;
__device__ __forceinline__ float slot_tmax(float tmax) { return tmax != tmax ? __uint_as_float(0x7FC00000u) : tmax; }

// slots of the batched form in use: B per level-1 node
__device__ __forceinline__ uint32_t batch_slots(const crsh_meta *meta, uint32_t B, uint32_t slot_cap)
{
    const uint64_t ns = meta->n_levels ? (uint64_t)meta->level_cnt[0] * B : 0u;
    return (uint32_t)(ns < slot_cap ? ns : slot_cap);
}

// A ray's slot: origin and tmax; direction and the |D| of the filter's T;
// o x D and the |o||D| of T, or FLT_KEEP in its place.
__device__ __forceinline__ void put_slot(const hit_slots_ws &hs, uint32_t p, f3 O, f3 D, f3 centre, float tmax)
{
    const f3 oc = O - centre;
    const float lo = len(oc) + FLT_TINY, ld = len(D);
    const bool ok = lo <= FLT_LONG && ld <= FLT_LONG && ld >= FLT_SHORT;
    const f3 M = cross(oc, D);
    hs.org[p] = make_float4(O.x, O.y, O.z, tmax);
    hs.dir[p] = make_float4(D.x, D.y, D.z, ok ? ld : 1.0f);
    hs.mom[p] = make_float4(M.x, M.y, M.z, ok ? lo * ld : FLT_KEEP);
}

// Triangles and ray slots packed, in one launch.  Plain form: slot s is sorted
// ray s.  Batched form: slot p = leaf * B + j holds ray j of level-1 node
// `leaf` (first ray and count as the build recorded them), or padding; every
// slot's closest-hit key starts at all ones.
template <bool BATCH>
__global__ void k_hit_pack(tri_verts V, uint32_t m, hit_tris_ws tri, sorted_rays R, const crsh_meta *meta,
                           uint32_t ray_cap, uint32_t B, batch_dev bd, hit_slots_ws hs)
{
    const uint32_t stride = gridDim.x * blockDim.x, gid = blockIdx.x * blockDim.x + threadIdx.x;
    const f3 centre = filter_centre(V, m);
    const uint32_t n = min(meta->n_rays, ray_cap);
    const uint32_t ns = BATCH ? batch_slots(meta, B, hs.slots) : n;
    for (uint32_t p = gid; p < ns; p += stride) {
        uint32_t s = p;
        bool ok = true;
        if constexpr (BATCH) {
            const uint32_t leaf = p / B;
            const uint32_t j = p - leaf * B;
            const uint32_t info = bd.node_info[leaf];
            s = bd.node_first[leaf] + j;
            ok = j < (info & INFO_COUNT_MASK) && s < n && info >> INFO_FRAME_SHIFT < bd.n_frames;
            hs.keys[p] = ~0ull;
        }
        if (ok) {
            put_slot(hs, p, mk(R.ox[s], R.oy[s], R.oz[s]), mk(R.dx[s], R.dy[s], R.dz[s]), centre,
                     BATCH ? slot_tmax(R.tmax[s]) : R.tmax[s]);
        } else {
            hs.org[p] = make_float4(0.0f, 0.0f, 0.0f, __uint_as_float(PAD_SLOT));
            hs.dir[p] = make_float4(0.0f, 0.0f, 0.0f, -1.0f);
            hs.mom[p] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
    }
    for (uint32_t t = gid; t <= m; t += stride) put_tri(V, t, m, centre, tri);
}

// Slots in use: the plain form's sorted rays, or B per level-1 node.  PACKED:
// the level-1 pairs are packed words in ptri (node above the low
// CRSH_PACKED_TRI_BITS, triangle minus tri_base below; pnode unused).
// Batched form: the build's per-node record of a leaf (bd.node_info) holds
// its ray count and frame, and the frame its interval start.
//
// Fused and listed: the level-1 pairs are not stored; they are the children that
// the pass bits of the level-2 pairs keep, placed in the leaf runs from there.
//
// A workgroup takes a chunk of consecutive pairs.  Pairs of one top-level
// node name a few hundred leaves in triangle order, so a chunk holds many
// pairs of each of its leaves: they are counted per leaf with LDS atomics
// (HIT_BINS bins: the leaves from the smallest on or, where they span more, the
// leaves that have pairs, numbered by a bitmap; what then has no bin waits for
// another round over the chunk), scanned, and the triangle ids scattered to
// their leaf's run in LDS, cut into blocks of at most G triangles (G: the
// bundle rounded up to a power of two, at least 4) -- the whole blocks
// first, then the leaves' remainders.  A wave takes 64 / G blocks at a time:
// lane j of a group of G holds ray j of the block's leaf and triangle j of
// the block, and each 4x4x1 matrix instruction tests the group's G rays
// against four of its triangles (the A operand broadcast from the lanes that
// hold them), 11 of them per 256 tests: six products for 2 a - det, three
// for det, two for T (see put_tri).  What the filter lets through --
// (triangle, slot) items -- is queued in LDS and goes through the test as
// written 64 at a time, so the division and the rest run on full waves and
// only for the few percent of the tests whose u can pass (more where the filter's
// error bound is large next to the triangles: see there).  Every count is exact:
// tests are counted per leaf, u and u-v passes by the exact test.
//
// Measured (whole stage, 881.7 M level-1 pairs and 14.1 G tests of a 1920x1080
// frame, B = 16): 18.2 ms with one lane per (pair, ray) and no matrix
// instructions, 7.8 ms so (1024x1024 reflections, 1.57 G tests, 2.00 to 1.14 ms,
// bounce rays of a 512x512 frame 5.6 to 2.1, 24 frames batched 9.5 to 4.3).  97 % of the matrix work is on real pairs.
// The vector L1 is busiest (three 16-byte reads of a triangle's entry per
// pair), then vector issue.  On the same pairs: chunks of 8,192 pairs in 512
// threads 8.2 ms, of 2,048 10.0 ms; reading a step ahead 8.4 ms (registers);
// triangle entries through LDS (a third of the L1 accesses, but more
// instructions and fewer workgroups) 8.3 ms; the filter's outcome as wave masks
// instead of shifted sign bits 9.4 ms.
// Where a top-level node has more leaves than there are bins, a chunk's pairs
// still name few of them (256 of 12,700 spanned on average, 128x72 mixed rays, 2 to
// a leaf, merge factor 4, 8 levels): in windows of 1,024 leaves it was read 7
// times, 332 us (whole stage); by the leaves that have pairs once, 179, and 161
// with a lane per (pair, ray).
// Where a chunk has at most 256 leaves, each has several bins and the threads of
// those cut its blocks.  With one bin a leaf, and its one thread to cut up to 1,024
// blocks, pairs of few leaves took longest: 128x72 mixed rays, 4 to a leaf, 24 M
// pairs, 4 leaves below a top node 372 us where 1,024 took 150; so 171 and 158.
// Fused (640x360 mixed rays, 144 M level-2 pairs, 2.8 G tests): 5.4 ms with a
// lane per (child, ray), 1.85 ms so.  A chunk of 2,048 level-2 pairs has 2,500
// children there; 1,536 1.96 ms, 1,792 1.91, 2,560 2.17, 3,072 2.18 (more
// chunks overflow and are taken in halves); parts of what is expected to fit
// instead of equal ones 2.06 (a small rest each).
// Listed (merge factors above 4: about one of 16 children kept, here and there
// all), 256x256 reflections, bundle 2 of 16 nodes, 4 levels, whole call: 4.4 ms
// with every lane at its own children, 2.9 so, 2.8 with a lane per (child, ray);
// of 72x48 mixed rays 1.72, 1.10 and 1.01, bundle 16 of 8 2.29, 2.30 and 3.91.
constexpr uint32_t HIT_THREADS = 256;
constexpr uint32_t HIT_WAVES = HIT_THREADS / WAVE;
constexpr uint32_t HIT_PPT = 16;                            // pairs per thread of a chunk
constexpr uint32_t HIT_CHUNK = HIT_THREADS * HIT_PPT;       // most pairs of a chunk
constexpr uint32_t HIT_MIN_CHUNK = 64;                      // fewest
constexpr uint32_t HIT_BPT = 4;                             // leaf bins per thread
constexpr uint32_t HIT_BINS = HIT_THREADS * HIT_BPT;        // leaves binned per round
constexpr uint32_t HIT_SPAN = 1u << 15;                     // leaves that a round's bins can lie in
constexpr uint32_t HIT_COPIES = 8;                          // most bins of a leaf, as a power of two
constexpr uint32_t HIT_QUEUE = 128;                         // queued items of a wave
// registers for 5 workgroups per compute unit, 4 for the smallest groups (their
// block words take the LDS of more)
constexpr int hit_waves_per_simd(int lg) { return lg > 2 ? 5 : 4; }
// block word: first triangle (12 bits), triangles - 1 (5 bits), leaf from the round's first on (15 bits)
static_assert(HIT_CHUNK <= 1u << 12 && HIT_SPAN <= 1u << 15 && CRSH_MAX_BUNDLE <= 32, "block word");
// bitmap of the leaves and the counts before its words, 16 bits each, in s_tri
constexpr uint32_t HIT_SPAN_WORDS = HIT_SPAN / 32;
constexpr uint32_t HIT_SPAN_WPT = HIT_SPAN_WORDS / HIT_THREADS;
static_assert(HIT_SPAN_WORDS + HIT_SPAN_WORDS / 2 <= HIT_CHUNK && HIT_SPAN_WPT * HIT_THREADS == HIT_SPAN_WORDS, "bitmap");

// What the pairs are.  Fused and listed: level-2 pairs and a pass bit per child
// (the level-1 pairs are never stored): pair q keeps child j (leaf first + j,
// first = node * F or the build's record) when bit q * nf + j of `mask` is set.
// Fused (nf <= 4): every thread walks the children of its pairs.  Listed: the
// children kept, few of many, are listed in LDS first, and a chunk with more than
// hit_later() of them -- where nodes are hardly ever culled, up to 32,768 -- is left,
// as tiles of HIT_TILE pairs, to another launch (`rest`, `n_rest`; deferred: this
// is that launch), so that no workgroup is long alone with one.
// parts: workgroups of the launch before, whose counts stay.
enum { HIT_STORED, HIT_PACKED, HIT_FUSED, HIT_LISTED };
struct fused_in {
    const uint32_t *mask;
    uint32_t nf, F, parts;
    uint32_t *rest, *n_rest;
    bool deferred;
};
constexpr uint32_t HIT_FUSED_PPT = 8;                   // level-2 pairs per thread of a chunk
constexpr uint32_t HIT_TILE = 256;                      // pairs of such a tile
static_assert(64 * HIT_FUSED_PPT % HIT_TILE == 0 && HIT_TILE >= LEVEL_TILE, "whole tiles, no more than counts");
// most children that a chunk takes in parts by itself.  Small groups have the most
// pairs per workgroup, and the longest waits: 72x48, bundle 2 of 8 nodes, 5 levels
// 1,043 us at 2 chunks, 1,151 at 3; 512x512, bundle 16 of 8 nodes, 4 levels 2,380
// at 2, 2,305 at 3 (whole calls)
__host__ __device__ constexpr uint32_t hit_later(int lg) { return (lg == 2 ? 2u : 3u) * HIT_CHUNK; }

typedef float mfma4 __attribute__((ext_vector_type(4)));

// p[q .. q + 3] of the first n, one load where all four are there (dword
// alignment is enough for it)
__device__ __forceinline__ void load4(const uint32_t *__restrict__ p, uint32_t q, uint32_t n, uint32_t *v)
{
    typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(4)));
    if (q + 4 <= n) {
        const u4 x = *(const u4 *)(p + q);
        v[0] = x.x, v[1] = x.y, v[2] = x.z, v[3] = x.w;
    } else {
        v[0] = q < n ? p[q] : 0u;
        v[1] = q + 1 < n ? p[q + 1] : 0u;
        v[2] = q + 2 < n ? p[q + 2] : 0u;
        v[3] = 0u;
    }
}

// The filter of triangles 4 Q .. 4 Q + 3 of every group against the group's
// rays: lane l gets, in element i, ray l's values for triangle 4 Q + i.
template <int LG, int Q>
__device__ __forceinline__ void filter4(const float4 &f0, const float4 &f1, const float4 &f2, const float4 &mo,
                                        const float4 &di, mfma4 &g, mfma4 &det, mfma4 &thr)
{
#define CRSH_MM(a, b, c) __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, LG - 2, Q, 0)
    const mfma4 z = {0.0f, 0.0f, 0.0f, 0.0f};
    g = CRSH_MM(f0.x, mo.x, z);
    det = CRSH_MM(f2.x, di.x, z);
    thr = CRSH_MM(f0.w, mo.w, z);
    g = CRSH_MM(f0.y, mo.y, g);
    det = CRSH_MM(f2.y, di.y, det);
    thr = CRSH_MM(f1.w, di.w, thr);
    g = CRSH_MM(f0.z, mo.z, g);
    det = CRSH_MM(f2.z, di.z, det);
    g = CRSH_MM(f1.x, di.x, g);
    g = CRSH_MM(f1.y, di.y, g);
    g = CRSH_MM(f1.z, di.z, g);
#undef CRSH_MM
}

// The filter of this lane's ray against its group's triangles 4 Q and on: one
// bit each, in order, shifted into rej, set if the triangle is surely
// rejected: the sign of T - (|2 a - det| - |det|) (meaningless for a ray
// marked FLT_KEEP, which the caller keeps).  cols: the lanes whose group has a
// triangle in their column.
template <int LG, int Q>
__device__ __forceinline__ void filter_all(const float4 &f0, const float4 &f1, const float4 &f2, const float4 &mo,
                                           const float4 &di, uint64_t cols, uint32_t &rej)
{
    constexpr uint32_t G = 1u << LG;
    // lanes 4 Q of every group
    constexpr uint64_t ONES = G == 4 ? 0x1111111111111111ull : G == 8 ? 0x0101010101010101ull
                            : G == 16 ? 0x0001000100010001ull : 0x0000000100000001ull;
    if constexpr (4 * Q < (int)G) {
        if ((cols & (ONES << (4 * Q))) != 0) {
            mfma4 g, det, thr;
            filter4<LG, Q>(f0, f1, f2, mo, di, g, det, thr);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float x = thr[i] - (fabsf(g[i]) - fabsf(det[i]));
                rej = __builtin_amdgcn_alignbit(rej, __float_as_uint(x), 31);
            }
            filter_all<LG, Q + 1>(f0, f1, f2, mo, di, cols, rej);
        } else {                    // no triangles left in any group
            rej = ~(~rej << (G - 4 * Q) % 32u);
        }
    }
}

template <int LG, bool BATCH, int IN>
__global__ __launch_bounds__(HIT_THREADS, hit_waves_per_simd(LG)) void k_hit(hit_slots_ws hs, const float4 *__restrict__ tri,
                                                     const float4 *__restrict__ ftri,
                                                     const uint32_t *__restrict__ ptri,
                                                     const uint32_t *__restrict__ pnode, uint64_t cap1, uint32_t B,
                                                     unsigned long long *keys, crsh_meta *meta, uint32_t m,
                                                     uint32_t tri_base, batch_dev bd, float t_min, uint32_t chunk_max,
                                                     fused_in fu)
{
    constexpr bool PACKED = IN == HIT_PACKED, LIST = IN == HIT_LISTED, FUSED = IN == HIT_FUSED || LIST;
    // pairs of a thread: children of a list as many as stored pairs
    constexpr uint32_t PPT = IN == HIT_FUSED ? HIT_FUSED_PPT : HIT_PPT;
    constexpr uint32_t G = 1u << LG;                // lanes, and triangles of a block, per group
    constexpr uint32_t GPW = WAVE / G;              // groups of a wave
    constexpr uint32_t NONE = 0xFFFFFFFFu;
    __shared__ __attribute__((aligned(8))) uint32_t s_tri[HIT_CHUNK];           // triangle ids, leaf by leaf
    __shared__ uint32_t s_binned[HIT_BINS + HIT_CHUNK / G + HIT_BINS];
    uint32_t *const s_cnt = s_binned;               // pairs per bin, then the bin's first place
    uint32_t *const s_blk = s_binned + HIT_BINS;    // blocks; first the leaves of the bins, if not consecutive
    static_assert(2 * HIT_CHUNK <= sizeof(s_binned) && HIT_FUSED_PPT * HIT_THREADS * 2 <= HIT_CHUNK, "fused lists");
    __shared__ uint32_t s_from;
    __shared__ uint2 s_queue[HIT_WAVES][HIT_QUEUE];
    __shared__ uint2 s_scan[HIT_WAVES], s_lohi[HIT_WAVES];
    __shared__ uint64_t s_red[3][HIT_WAVES];
    const uint32_t ns = BATCH ? batch_slots(meta, B, hs.slots) : min(meta->n_rays, hs.slots);
    uint64_t np = meta->n_levels > (FUSED ? 1u : 0u) ? meta->pairs[FUSED ? 1 : 0] : 0;
    np = np < cap1 ? np : cap1;
    const uint32_t off2 = FUSED ? meta->level_off[1] : 0u, np2 = FUSED ? meta->level_cnt[1] : 0u;
    // no slots, no tests
    const uint32_t last_leaf = ns ? (ns - 1u) / B : 0u;
    np = ns ? np : 0u;
    const uint32_t l = lane_id();
    const uint32_t j = l & (G - 1);
    const uint32_t wib = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const __amdgpu_buffer_rsrc_t org_r = make_rsrc(hs.org, (uint64_t)ns * 16u);
    const __amdgpu_buffer_rsrc_t dir_r = make_rsrc(hs.dir, (uint64_t)ns * 16u);
    const __amdgpu_buffer_rsrc_t mom_r = make_rsrc(hs.mom, (uint64_t)ns * 16u);
    const __amdgpu_buffer_rsrc_t ftri_r = make_rsrc(ftri, ((uint64_t)m + 1) * 48u);
    const __amdgpu_buffer_rsrc_t tri_r = make_rsrc(tri, (uint64_t)m * 48u);
    uint2 *const queue = s_queue[wib];
    uint32_t qn = 0;                                // items in the queue (wave-uniform)
    uint64_t tests = 0, upass = 0, uvpass = 0;      // tests: this thread's; the others: wave-wide

    // the test as written for one item a lane
    auto exact = [&](uint2 it, uint64_t live) {
        live &= ballot(it.x < m);                   // not a padding triangle
        const uint32_t ro = it.y * 16u, to = it.x * 48u;
        const float4 o4 = buf_load4(org_r, ro);
        const float4 d4 = buf_load4(dir_r, ro);
        const float4 ta = buf_load4(tri_r, to);
        const float4 tb = buf_load4(tri_r, to + 16u);
        const float tc = buf_load1(tri_r, to + 32u);
        float tm = t_min;
        if constexpr (BATCH) {
            const uint32_t info = ((live >> l) & 1u) ? bd.node_info[it.y / B] : 0u;
            const uint32_t f = info >> INFO_FRAME_SHIFT;
            tm = f < bd.n_frames ? bd.frames[f].t_min : 0.0f;
        }
        tri_t tr;
        tr.v0 = mk(ta.x, ta.y, ta.z);
        tr.e1 = mk(ta.w, tb.x, tb.y);
        tr.e2 = mk(tb.z, tb.w, tc);
        const f3 D = mk(d4.x, d4.y, d4.z);
        mt_head h;
        const uint64_t mm = mt_first_half(mk(o4.x, o4.y, o4.z), D, tr, h) & live;
        float th;
        uint64_t pu, puv, hit;
        mt_second_half(D, tm, o4.w, tr, h, th, pu, puv, hit);
        upass += (uint64_t)__popcll(pu & mm);
        uvpass += (uint64_t)__popcll(puv & mm);
        if (__builtin_amdgcn_inverse_ballot_w64(hit & mm)) atomicMin(&keys[it.y], hit_key(th, it.x));
    };

    // near-equal chunks in whole rounds of the grid, at most chunk_max pairs each
    const float rounds = ceilf((float)np / ((float)gridDim.x * (float)chunk_max));
    uint32_t cs = rounds > 0.0f ? (uint32_t)((float)np / (rounds * (float)gridDim.x)) + 1u : 1u;
    constexpr uint32_t UNIT = LIST ? HIT_TILE : HIT_MIN_CHUNK;
    cs = min(max((cs + UNIT - 1u) & ~(UNIT - 1u), UNIT), chunk_max);
    // pass bits of the four pairs from q on (q a multiple of 4), pair q + i in
    // the bits from i * nf on
    auto load_bits = [&](uint64_t q, uint2 &w, uint32_t &sh) {
        const uint64_t bit = q * fu.nf;
        w.x = fu.mask[bit >> 5];
        w.y = fu.nf > 8u ? fu.mask[(bit >> 5) + 1] : 0u;
        sh = (uint32_t)bit & 31u;
    };
    auto bits_of = [&](uint2 w, uint32_t sh, uint32_t i) {
        const uint32_t at = sh + i * fu.nf;
        return (at < 32u ? w.x >> at : w.y >> (at - 32u)) & ((1u << fu.nf) - 1u);
    };
    const bool deferred = LIST && fu.deferred;
    if (deferred) cs = HIT_TILE;
    const uint64_t chunks = deferred ? (np ? *fu.n_rest : 0u) : (np + cs - 1) / cs;
    for (uint64_t ci = blockIdx.x; ci < chunks; ci += gridDim.x) {
    const uint64_t chunk = (uint64_t)cs * (deferred ? fu.rest[ci] : ci);
    const uint32_t chunk_n = (uint32_t)min(np - chunk, (uint64_t)cs);
    // (once; fused: as many pairs at a time as have survivors that fit)
    for (uint32_t done = 0, cn; done < chunk_n; done += cn) {
        const uint64_t c0 = chunk + done;
        cn = chunk_n - done;
        bool later = false;
        if constexpr (FUSED) {
            // equal parts of the rest as long as the survivors do not fit
            // (those of 256 pairs always do)
            for (;;) {
                uint32_t kids = 0u;
#pragma unroll
                for (uint32_t k = 0; k < HIT_FUSED_PPT; k += 4) {
                    const uint32_t q = k * HIT_THREADS + 4 * threadIdx.x;
                    if (q >= cn) continue;
                    uint2 w;
                    uint32_t sh;
                    load_bits(c0 + q, w, sh);
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i) kids += q + i < cn ? (uint32_t)__popc(bits_of(w, sh, i)) : 0u;
                }
                kids = wave_reduce(kids, 0u, [](uint32_t a, uint32_t b) { return a + b; });
                if (l == 0) s_lohi[wib].x = kids;
                __syncthreads();
                kids = 0u;
#pragma unroll
                for (uint32_t w = 0; w < HIT_WAVES; ++w) kids += s_lohi[w].x;
                __syncthreads();                    // s_lohi is written again
                kids = __builtin_amdgcn_readfirstlane(kids);
                if (kids <= HIT_CHUNK) break;
                later = LIST && !deferred && kids > hit_later(LG);
                if (later) break;
                const uint32_t parts = (kids - 1u) / HIT_CHUNK + 1u;        // at least 2
                cn = ((cn - 1u) / parts + 64u) & ~63u;
            }
        }
        if (later) {
            const uint32_t n = (cn + HIT_TILE - 1u) / HIT_TILE;
            if (threadIdx.x == 0) s_from = atomicAdd(fu.n_rest, n);
            __syncthreads();
            if (threadIdx.x < n) fu.rest[s_from + threadIdx.x] = (uint32_t)(c0 / HIT_TILE) + threadIdx.x;
            __syncthreads();                        // s_from is written again
            continue;
        }
        uint32_t from = 0u;                         // first leaf not binned yet
        for (bool more = true; more;) {
            uint32_t tid = threadIdx.x;
            asm volatile("" : "+v"(tid));           // nothing of a round is kept over the next
            // my_leaf: the pair's leaf (fused: the first child of its node)
            uint32_t my_t[PPT], my_leaf[PPT], my_bits[IN == HIT_FUSED ? PPT : 1];
            uint32_t lo = NONE, hi = 0u;            // the leaves still to do: smallest and largest
            // pass bits of pair i of four, of the children that have rays (a pair
            // out of range has none); f: its first child
            auto kept = [&](uint32_t q, uint32_t t, uint32_t node, uint2 w, uint32_t sh, uint32_t i, uint32_t &f) {
                uint32_t b = q < cn && t < m && node < np2 ? bits_of(w, sh, i) : 0u;
                f = node * fu.F;
                if constexpr (BATCH) f = b ? bd.node_first[off2 + node] : 0u;
                return f <= last_leaf ? b & (uint32_t)((1ull << min(last_leaf - f + 1u, 16u)) - 1ull) : 0u;
            };
            if constexpr (LIST) {
                // the children that the pass bits keep, listed in LDS (pair of
                // the chunk, child) with the pairs beside them (triangle, first
                // child), so that the lanes share them evenly
                uint2 *const par = (uint2 *)s_tri;
                uint16_t *const item = (uint16_t *)s_binned;
                uint32_t bits[HIT_FUSED_PPT], n = 0u;
                __syncthreads();                    // the round before is done with these
#pragma unroll
                for (uint32_t k = 0; k < HIT_FUSED_PPT; k += 4) {
                    const uint32_t q = k * HIT_THREADS + 4 * tid;
                    uint32_t t[4], node[4], sh = 0u;
                    load4(ptri + c0, q, cn, t);
                    load4(pnode + c0, q, cn, node);
                    uint2 w = make_uint2(0u, 0u);
                    if (q < cn) load_bits(c0 + q, w, sh);
#pragma unroll
                    for (uint32_t i = 0; i < 4; ++i) {
                        uint32_t f;
                        bits[k + i] = kept(q + i, t[i], node[i], w, sh, i, f);
                        n += (uint32_t)__popc(bits[k + i]);
                        par[q + i] = make_uint2(t[i], f);
                    }
                }
                uint32_t at = wave_scan_dpp(n), all = 0u;
                if (l == WAVE - 1) s_scan[wib].x = at;
                at -= n;
                __syncthreads();
#pragma unroll
                for (uint32_t w = 0; w < HIT_WAVES; ++w) {
                    const uint32_t v = s_scan[w].x;
                    at += w < wib ? v : 0u;
                    all += v;
                }
#pragma unroll
                for (uint32_t k = 0; k < HIT_FUSED_PPT; ++k) {
                    const uint32_t q = k / 4 * 4 * HIT_THREADS + 4 * tid + k % 4;
                    for (uint32_t b = bits[k]; b != 0u; b &= b - 1u)
                        item[at++] = (uint16_t)(q << 4 | (uint32_t)__builtin_ctz(b));
                }
                __syncthreads();
#pragma unroll
                for (uint32_t k = 0; k < HIT_PPT; ++k) {
                    const uint32_t i = k * HIT_THREADS + tid;
                    const uint32_t it = item[i < all ? i : 0u];
                    const uint2 p = par[it >> 4];
                    const uint32_t leaf = p.y + (it & 15u);
                    const bool ok = i < all && leaf >= from;
                    my_t[k] = p.x;
                    hi = ok ? max(hi, leaf) : hi;
                    my_leaf[k] = ok ? leaf : NONE;
                    lo = min(lo, my_leaf[k]);
                }
                __syncthreads();                    // s_cnt is cleared
            } else {
#pragma unroll
                for (uint32_t k = 0; k < PPT; k += 4) {     // four consecutive pairs a load
                    const uint32_t q = k * HIT_THREADS + 4 * tid;
                    load4(ptri + c0, q, cn, &my_t[k]);
                    if constexpr (!PACKED) load4(pnode + c0, q, cn, &my_leaf[k]);
                    if constexpr (FUSED) {
                        uint2 w = make_uint2(0u, 0u);
                        uint32_t sh = 0u;
                        if (q < cn) load_bits(c0 + q, w, sh);
#pragma unroll
                        for (uint32_t i = 0; i < 4; ++i) {
                            uint32_t f, b = kept(q + i, my_t[k + i], my_leaf[k + i], w, sh, i, f);
                            b = f < from ? b >> min(from - f, 31u) << min(from - f, 31u) : b;
                            my_bits[k + i] = b;
                            my_leaf[k + i] = f;
                            lo = b ? min(lo, f + (uint32_t)__builtin_ctz(b)) : lo;
                            hi = b ? max(hi, f + 31u - (uint32_t)__builtin_clz(b)) : hi;
                        }
                    }
                }
                if constexpr (!FUSED)
#pragma unroll
                for (uint32_t k = 0; k < PPT; ++k) {
                    const uint32_t q = k / 4 * 4 * HIT_THREADS + 4 * tid + k % 4;
                    if constexpr (PACKED) {
                        my_leaf[k] = my_t[k] >> CRSH_PACKED_TRI_BITS;
                        my_t[k] = tri_base + (my_t[k] & ((1u << CRSH_PACKED_TRI_BITS) - 1u));
                    }
                    // a pair out of range has no tests
                    const bool ok = q < cn && my_t[k] < m && my_leaf[k] <= last_leaf && my_leaf[k] >= from;
                    hi = ok ? max(hi, my_leaf[k]) : hi;
                    my_leaf[k] = ok ? my_leaf[k] : NONE;
                    lo = min(lo, my_leaf[k]);
                }
            }
            lo = wave_reduce(lo, NONE, [](uint32_t a, uint32_t b) { return min(a, b); });
            hi = wave_reduce(hi, 0u, [](uint32_t a, uint32_t b) { return max(a, b); });
            if (l == 0) s_lohi[wib] = make_uint2(lo, hi);
#pragma unroll
            for (uint32_t k = 0; k < HIT_BPT; ++k) s_cnt[tid + k * HIT_THREADS] = 0u;
            __syncthreads();
#pragma unroll
            for (uint32_t w = 0; w < HIT_WAVES; ++w) {
                const uint2 v = s_lohi[w];
                lo = min(lo, v.x);
                hi = max(hi, v.y);
            }
            const uint32_t base = __builtin_amdgcn_readfirstlane(lo);
            hi = __builtin_amdgcn_readfirstlane(hi);
            const bool wide = base != NONE && hi - base >= HIT_BINS;
            uint32_t used = min(hi - base + 1u, HIT_BINS);      // bins in use
            uint32_t leaves = 0u;                               // (wide) that have pairs
            more = false;
            // the leaves counted from the round's first on
#pragma unroll
            for (uint32_t k = 0; k < PPT; ++k)
                my_leaf[k] = IN == HIT_FUSED || my_leaf[k] != NONE ? my_leaf[k] - base : NONE;
            // wide: the bins are the leaves that have pairs, in order, and
            // my_leaf becomes the bin (fused: the first child in the low 15
            // bits, then a bit for each child that has a bin, then the first bin)
            if (wide) {
                if constexpr (IN == HIT_FUSED) {
                    // first children before the round's first: those bits are clear
#pragma unroll
                    for (uint32_t k = 0; k < PPT; ++k) {
                        const uint32_t sh = 0u - my_leaf[k] < 4u ? 0u - my_leaf[k] : 0u;
                        my_bits[k] >>= sh;
                        my_leaf[k] += sh;
                    }
                }
                uint32_t *const map = s_tri;
                uint16_t *const before = (uint16_t *)(s_tri + HIT_SPAN_WORDS);
#pragma unroll
                for (uint32_t k = 0; k < HIT_SPAN_WPT; ++k) map[tid + k * HIT_THREADS] = 0u;
                __syncthreads();
#pragma unroll
                for (uint32_t k = 0; k < PPT; ++k) {
                    const uint32_t w = my_leaf[k] / 32u;
                    if constexpr (IN == HIT_FUSED) {
                        const uint64_t b = (uint64_t)my_bits[k] << (my_leaf[k] & 31u);
                        if ((uint32_t)b != 0u && w < HIT_SPAN_WORDS) atomicOr(&map[w], (uint32_t)b);
                        if (b >> 32 != 0u && w < HIT_SPAN_WORDS - 1u) atomicOr(&map[w + 1], (uint32_t)(b >> 32));
                    } else if (w < HIT_SPAN_WORDS) {
                        atomicOr(&map[w], 1u << (my_leaf[k] & 31u));
                    }
                }
                __syncthreads();
                uint32_t n = 0u, own[HIT_SPAN_WPT];
#pragma unroll
                for (uint32_t k = 0; k < HIT_SPAN_WPT; ++k) {
                    own[k] = map[HIT_SPAN_WPT * tid + k];
                    n += (uint32_t)__popc(own[k]);
                }
                uint32_t bin = wave_scan_dpp(n);
                if (l == WAVE - 1) s_scan[wib].x = bin;
                bin -= n;
                __syncthreads();
#pragma unroll
                for (uint32_t w = 0; w < HIT_WAVES; ++w) {
                    const uint32_t v = s_scan[w].x;
                    bin += w < wib ? v : 0u;
                    leaves += v;
                }
                leaves = __builtin_amdgcn_readfirstlane(leaves);
#pragma unroll
                for (uint32_t k = 0; k < HIT_SPAN_WPT; ++k) {
                    before[HIT_SPAN_WPT * tid + k] = (uint16_t)bin;
                    bin += (uint32_t)__popc(own[k]);
                }
                __syncthreads();
                used = min(leaves, HIT_BINS);
#pragma unroll
                for (uint32_t k = 0; k < PPT; ++k) {
                    const uint32_t w = min(my_leaf[k] / 32u, HIT_SPAN_WORDS - 1u), sh = my_leaf[k] & 31u;
                    const uint32_t bits = map[w], b = before[w] + (uint32_t)__popc(bits & ((1u << sh) - 1u));
                    const bool in = my_leaf[k] < HIT_SPAN;
                    // (the leaf of a bin is put down by all its pairs)
                    if constexpr (IN == HIT_FUSED) {
                        const uint32_t up = w + 1 < HIT_SPAN_WORDS ? map[w + 1] : 0u;
                        const uint32_t has = (uint32_t)(((uint64_t)up << 32 | bits) >> sh) & 15u;
                        my_bits[k] = in ? my_bits[k] & has : 0u;
                        uint32_t at = b;
#pragma unroll
                        for (uint32_t c = 0; c < 4; ++c) {
                            if ((my_bits[k] >> c & 1u) != 0u && at < HIT_BINS) s_blk[at] = my_leaf[k] + c;
                            if ((my_bits[k] >> c & 1u) != 0u && at == HIT_BINS) s_from = base + my_leaf[k] + c;
                            at += has >> c & 1u;
                        }
                        my_leaf[k] = (my_leaf[k] & (HIT_SPAN - 1u)) | has << 15 | b << 19;
                    } else {
                        if (in && b < HIT_BINS) s_blk[b] = my_leaf[k];
                        if (in && b == HIT_BINS) s_from = base + my_leaf[k];
                        my_leaf[k] = in ? b : NONE;
                    }
                    if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);     // few in flight: registers
                }
            }
            // few leaves: 2^copies bins each, by thread
            const uint32_t copies = used > HIT_THREADS ? 0u : min((uint32_t)__builtin_clz((used - 1u) | 1u) - 22u, HIT_COPIES);
            const uint32_t copy = tid & ((1u << copies) - 1u), bins = HIT_BINS >> copies;
            // fused: body(bin, pair) for every child that has a bin
            auto children = [&](auto body) {
                auto each = [&](auto bin_of) {
                    for (uint32_t c = 0; c < fu.nf; ++c)
#pragma unroll
                        for (uint32_t k = 0; k < PPT; ++k) {
                            const uint32_t bin = bin_of(my_leaf[k], c);
                            if ((my_bits[k] >> c & 1u) != 0u && bin < bins) body(bin << copies | copy, k);
                        }
                };
                if (wide)
                    each([](uint32_t v, uint32_t c) { return (v >> 19) + (uint32_t)__popc((v >> 15) & ((1u << c) - 1u)); });
                else
                    each([](uint32_t v, uint32_t c) { return v + c; });
            };
            // pairs per leaf; each pair's bin and its place in the bin's run
            // (fused: the place is taken when the triangle is put there)
            if constexpr (IN == HIT_FUSED)
                children([&](uint32_t bin, uint32_t) { atomicAdd(&s_cnt[bin], 1u); });
            else
#pragma unroll
            for (uint32_t k = 0; k < PPT; ++k) {
                const bool ok = my_leaf[k] < bins;
                const uint32_t bin = my_leaf[k] << copies | copy;
                my_leaf[k] = NONE;
                if (ok) my_leaf[k] = bin | atomicAdd(&s_cnt[bin], 1u) * HIT_BINS;
            }
            __syncthreads();
            if (wide) {                 // what has no bin waits
                more = leaves > HIT_BINS || hi - base >= HIT_SPAN;
                from = leaves > HIT_BINS ? __builtin_amdgcn_readfirstlane(s_from) : base + HIT_SPAN;
            }
            // places, whole blocks and remainders of the leaves
            uint32_t nfull = 0u, nblk = 0u;
            auto count_tests = [&](uint32_t leaf, uint32_t pairs) {
                uint32_t rays = min(B, ns - (base + leaf) * B);
                if constexpr (BATCH) rays = min(rays, bd.node_info[base + leaf] & INFO_COUNT_MASK);
                tests += (uint64_t)pairs * rays;
            };
            // exclusive sums over the workgroup of x and y; nfull and nblk: the
            // totals of y, and of y and the high half of x
            auto sums = [&](uint32_t &x, uint32_t &y) {
                const uint32_t x0 = x, y0 = y;
                x = wave_scan_dpp(x);
                y = wave_scan_dpp(y);
                if (l == WAVE - 1) s_scan[wib] = make_uint2(x, y);
                x -= x0;
                y -= y0;
                __syncthreads();
                nfull = nblk = 0u;
#pragma unroll
                for (uint32_t w = 0; w < HIT_WAVES; ++w) {
                    const uint2 v = s_scan[w];
                    x += w < wib ? v.x : 0u;
                    y += w < wib ? v.y : 0u;
                    nfull += v.y;
                    nblk += v.x >> 16;
                }
                nfull = __builtin_amdgcn_readfirstlane(nfull);
                nblk = __builtin_amdgcn_readfirstlane(nblk) + nfull;
            };
            if (copies) {
                // a thread's four bins are of one leaf; it cuts the blocks that
                // begin at their places, and thread x the remainder of leaf x
                const uint32_t my_id = wide ? s_blk[tid] : tid;
                uint32_t c[HIT_BPT], at = 0u, ex_f = 0u;
#pragma unroll
                for (uint32_t k = 0; k < HIT_BPT; ++k) {
                    c[k] = s_cnt[HIT_BPT * tid + k];
                    at += c[k];
                }
                sums(at, ex_f);
                const uint32_t my0 = at;
#pragma unroll
                for (uint32_t k = 0; k < HIT_BPT; ++k) {
                    s_cnt[HIT_BPT * tid + k] = at;
                    at += c[k];
                }
                const uint32_t my1 = at;
                if (tid == HIT_THREADS - 1) s_from = my1;       // the chunk's pairs
                __syncthreads();
                const uint32_t all = s_from, first = tid < bins ? s_cnt[tid << copies] : all;
                const uint32_t n = (tid + 1u < bins ? s_cnt[(tid + 1u) << copies] : all) - first;
                uint32_t part = n % G != 0u ? 1u << 16 : 0u;
                ex_f = n / G;
                sums(part, ex_f);
                if (tid < bins) {
                    s_tri[tid] = ex_f;
                    s_tri[HIT_THREADS + tid] = first | (n / G) << 16;
                    s_tri[2 * HIT_THREADS + tid] = my_id;
                }
                if (n) count_tests(my_id, n);
                if (n % G) s_blk[nfull + (part >> 16)] = (first + n / G * G) | (n % G - 1) << 12 | my_id << 17;
                __syncthreads();
                const uint32_t x = (HIT_BPT * tid) >> copies, f = s_tri[HIT_THREADS + x], to = s_tri[x];
                const uint32_t leaf_first = f & 0xFFFFu, leaf_id = s_tri[2 * HIT_THREADS + x];
                for (uint32_t k = (my0 - leaf_first + G - 1) / G; k < f >> 16 && leaf_first + k * G < my1; ++k)
                    s_blk[to + k] = (leaf_first + k * G) | (G - 1) << 12 | leaf_id << 17;
            } else {
                uint32_t c[HIT_BPT], leaf[HIT_BPT], ex_cp = 0u, ex_f = 0u;
#pragma unroll
                for (uint32_t k = 0; k < HIT_BPT; ++k) {
                    const uint32_t bin = HIT_BPT * tid + k;
                    leaf[k] = wide ? s_blk[bin] : bin;
                    c[k] = s_cnt[bin];
                    ex_cp += c[k] | (c[k] % G != 0u ? 1u << 16 : 0u);
                    ex_f += c[k] / G;
                }
                sums(ex_cp, ex_f);
                uint32_t first = ex_cp & 0xFFFFu, part = nfull + (ex_cp >> 16);
#pragma unroll
                for (uint32_t k = 0; k < HIT_BPT; ++k) {
                    s_cnt[HIT_BPT * tid + k] = first;
                    if (c[k] == 0u) continue;
                    uint32_t rest = c[k];
                    for (; rest >= G; rest -= G, first += G) s_blk[ex_f++] = first | (G - 1) << 12 | leaf[k] << 17;
                    if (rest) s_blk[part++] = first | (rest - 1) << 12 | leaf[k] << 17;
                    first += rest;
                    count_tests(leaf[k], c[k]);
                }
            }
            __syncthreads();
            if constexpr (IN == HIT_FUSED)
                children([&](uint32_t bin, uint32_t k) { s_tri[atomicAdd(&s_cnt[bin], 1u)] = my_t[k]; });
            else
#pragma unroll
            for (uint32_t k = 0; k < PPT; ++k)
                if (my_leaf[k] != NONE) s_tri[s_cnt[my_leaf[k] % HIT_BINS] + my_leaf[k] / HIT_BINS] = my_t[k];
            __syncthreads();
            for (uint32_t b0 = wib * GPW; b0 < nblk; b0 += HIT_WAVES * GPW) {
                const uint32_t bi = b0 + l / G;
                const uint32_t e = s_blk[bi < nblk ? bi : 0u];
                const uint32_t cnt = bi < nblk ? ((e >> 12) & 31u) + 1u : 0u;
                const uint32_t slot = (base + (e >> 17)) * B + j;
                const uint32_t t = j < cnt ? s_tri[(e & 0xFFFu) + j] : m;
                const uint64_t cols = ballot(j < cnt);
                const float4 f0 = buf_load4(ftri_r, t * 48u);
                const float4 f1 = buf_load4(ftri_r, t * 48u + 16u);
                const float4 f2 = buf_load4(ftri_r, t * 48u + 32u);
                const float4 mo = buf_load4(mom_r, slot * 16u);
                const float4 di = buf_load4(dir_r, slot * 16u);
                // this lane's ray against the block's G triangles: bit G - 1 - c
                // set if triangle c is rejected
                uint32_t rej = 0u;
                filter_all<LG, 0>(f0, f1, f2, mo, di, cols, rej);
                // the columns kept, one of every lane at a time
                rej = mo.w == FLT_KEEP ? 0u : rej;
                uint32_t kept = j < B && slot < ns && cnt != 0u ? ~rej & (uint32_t)((1ull << G) - 1ull) : 0u;
                for (uint64_t k; (k = ballot(kept != 0u)) != 0;) {
                    const uint32_t c = G - 32u + (uint32_t)__builtin_clz(kept | 1u);
                    const uint32_t tid = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(((l & ~(G - 1)) + (c & (G - 1))) * 4u), (int)t);
                    if (kept != 0u) queue[qn + rank_below(k)] = make_uint2(tid, slot);
                    kept &= ~(1u << (G - 1 - (c & (G - 1))));
                    qn += (uint32_t)__popcll(k);
                    if (qn >= WAVE) {
                        __builtin_amdgcn_wave_barrier();
                        const uint2 it = queue[l], rest = queue[WAVE + l];
                        __builtin_amdgcn_wave_barrier();
                        qn -= WAVE;
                        if (l < qn) queue[l] = rest;
                        __builtin_amdgcn_wave_barrier();
                        exact(it, ~0ull);
                    }
                }
            }
        }
    }
    }
    if (qn) {
        __builtin_amdgcn_wave_barrier();
        const uint2 it = queue[l];
        exact(l < qn ? it : make_uint2(m, 0u), (1ull << qn) - 1ull);
    }
    // this workgroup's counts; k_hit_final adds them up (atomics of every
    // workgroup on three words would take longer than a small frame's tests)
    tests = wave_sum(tests);
    if (l == 0) {
        s_red[0][wib] = tests;
        s_red[1][wib] = upass;
        s_red[2][wib] = uvpass;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        uint64_t tot = 0;
        for (uint32_t w = 0; w < HIT_WAVES; ++w) tot += s_red[threadIdx.x][w];
        uint64_t *const part = &hs.part[3 * blockIdx.x + threadIdx.x];
        *part = tot + (FUSED && blockIdx.x < fu.parts ? *part : 0u);
    }
}

struct hit_out {
    int32_t *tri;
    float *t, *u, *v;
};

// Batched form: the key of sorted ray s is its slot's (all of a call's tests go
// there, and a batch starts with no hits), and is left in tkey[s] as in the plain
// form.
template <bool BATCH>
__global__ void k_hit_final(sorted_rays R, const float4 *__restrict__ tri, const uint32_t *__restrict__ sorted_ids,
                            float t_min0, unsigned long long *tkey, const unsigned long long *__restrict__ keys,
                            uint32_t B, uint32_t slot_cap, hit_out out, crsh_meta *meta, uint32_t ray_cap,
                            uint32_t m, batch_dev bd, const uint64_t *part, uint32_t n_part)
{
    // the counts of k_hit's workgroups, by the first of this grid
    if (blockIdx.x == 0 && n_part) {
        __shared__ uint64_t s_red[3][256 / WAVE];
        uint64_t c[3] = {0, 0, 0};
        for (uint32_t i = threadIdx.x; i < n_part; i += blockDim.x)
            for (uint32_t k = 0; k < 3; ++k) c[k] += part[3 * i + k];
        for (uint32_t k = 0; k < 3; ++k) {
            c[k] = wave_sum(c[k]);
            if (lane_id() == 0) s_red[k][threadIdx.x / WAVE] = c[k];
        }
        __syncthreads();
        if (threadIdx.x < 3) {
            uint64_t tot = 0;
            for (uint32_t w = 0; w < 256 / WAVE; ++w) tot += s_red[threadIdx.x][w];
            uint64_t *const dst = threadIdx.x == 0 ? &meta->final_tests
                                : threadIdx.x == 1 ? &meta->final_u_pass : &meta->final_uv_pass;
            if (tot) *dst += tot;
        }
    }
    const uint32_t n = min(meta->n_rays, ray_cap);
    const uint32_t ns = BATCH ? batch_slots(meta, B, slot_cap) : 0u;
    for (uint32_t s = blockIdx.x * blockDim.x + threadIdx.x; s < n; s += gridDim.x * blockDim.x) {
        unsigned long long key = BATCH ? ~0ull : tkey[s];
        const uint32_t id = sorted_ids[s];
        if (id >= ray_cap) continue;    // ids come from the sort: never taken
        float t_min = t_min0;
        if constexpr (BATCH) {
            const uint32_t f = min(bd.ray_frame[id], bd.n_frames - 1);
            t_min = bd.frames[f].t_min;
            const uint32_t rb = bd.fm[f].ray_begin;
            const uint64_t p = (uint64_t)bd.fm[f].level_base[0] * B + (s - rb);
            if (s >= rb && p < ns) key = keys[p];
            tkey[s] = key;
        }
        int32_t best = -1;
        float th = 0.0f, uh = 0.0f, vh = 0.0f;
        if (key != ~0ull && (uint32_t)(key & 0xFFFFFFFFull) < m) {
            const uint32_t t = (uint32_t)(key & 0xFFFFFFFFull);
            const f3 O = mk(R.ox[s], R.oy[s], R.oz[s]);
            const f3 D = mk(R.dx[s], R.dy[s], R.dz[s]);
            if (moller_trumbore(O, D, t_min, R.tmax[s], load_tri(tri, t), th, uh, vh)) {
                best = (int32_t)t;
            } else {                     // cannot happen: same inputs, same operations
                best = (int32_t)t;
                th = hit_key_t(key);
            }
        }
        out.tri[id] = best;
        out.t[id] = th;
        out.u[id] = uh;
        out.v[id] = vh;
    }
}

__global__ void k_tkey_fill(unsigned long long *tkey, uint32_t n)
{
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) tkey[i] = ~0ull;
}

}  // namespace crsh

using namespace crsh;

extern "C" crsh_status crsh_hits_reset(crsh_hits *hits, hipStream_t stream)
{
    if (!hits || !hits->tkey) {
        set_error("crsh_hits_reset: NULL argument");
        return CRSH_ERR_INVALID;
    }
    uint32_t g = std::min<uint32_t>((hits->capacity + 255) / 256, 4096);
    if (g == 0) g = 1;
    k_tkey_fill<<<g, 256, 0, stream>>>(hits->tkey, hits->capacity);
    return hip_check(hipGetLastError(), "crsh_hits_reset launch");
}

namespace crsh {

void hit_pack_launch(const crsh_scene *scene, const hit_tris_ws &tri, const crsh_rays *sorted,
                     const hit_slots_ws &hs, int32_t bundle, const crsh_meta *meta, const batch_dev *bd,
                     hipStream_t stream)
{
    tri_verts V;
    for (int k = 0; k < 9; ++k) V.v[k] = scene->v[k];
    const sorted_rays S{sorted->ox, sorted->oy, sorted->oz, sorted->dx, sorted->dy, sorted->dz, sorted->tmax};
    const uint32_t items = std::max(hs.slots, scene->m + 1);
    const uint32_t g = std::min<uint32_t>((items + 255) / 256, 4096);
    if (bd)
        k_hit_pack<true><<<g, 256, 0, stream>>>(V, scene->m, tri, S, meta, sorted->capacity, (uint32_t)bundle, *bd, hs);
    else
        k_hit_pack<false><<<g, 256, 0, stream>>>(V, scene->m, tri, S, meta, sorted->capacity, (uint32_t)bundle,
                                                 batch_dev{}, hs);
}

template <int LG, int IN>
static uint32_t k_hit_launch(const hit_slots_ws &hs, const hit_tris_ws &tri, const crsh_pairs *pairs, uint32_t B,
                             crsh_hits *hits, crsh_meta *meta, uint32_t m, uint32_t tri_base, const batch_dev *bd,
                             float t_min, uint32_t chunk, const fused_in &fu, hipStream_t stream)
{
    // one round of resident workgroups, at most one per smallest chunk
    const uint64_t want = std::min<uint64_t>(
        std::max<uint64_t>((pairs->capacity + HIT_MIN_CHUNK - 1) / HIT_MIN_CHUNK, 1), HIT_MAX_GRID);
    uint32_t g;
    if constexpr (IN != HIT_PACKED) {
        if (bd) {
            g = resident_grid((const void *)k_hit<LG, true, IN>, HIT_THREADS, want);
            k_hit<LG, true, IN><<<g, HIT_THREADS, 0, stream>>>(hs, tri.tri, tri.ftri, pairs->tri, pairs->node,
                                                               pairs->capacity, B, hs.keys, meta, m, 0u, *bd, 0.0f,
                                                               chunk, fu);
            return g;
        }
    }
    g = resident_grid((const void *)k_hit<LG, false, IN>, HIT_THREADS, want);
    k_hit<LG, false, IN><<<g, HIT_THREADS, 0, stream>>>(hs, tri.tri, tri.ftri, pairs->tri, pairs->node,
                                                        pairs->capacity, B, hits->tkey, meta, m, tri_base,
                                                        batch_dev{}, t_min, chunk, fu);
    return g;
}

template <int IN>
static uint32_t k_hit_launch(const hit_slots_ws &hs, const hit_tris_ws &tri, const crsh_pairs *pairs, uint32_t B,
                             crsh_hits *hits, crsh_meta *meta, uint32_t m, uint32_t tri_base, const batch_dev *bd,
                             float t_min, uint32_t chunk, const fused_in &fu, hipStream_t stream)
{
#define CRSH_HIT(LG) \
    return k_hit_launch<LG, IN>(hs, tri, pairs, B, hits, meta, m, tri_base, bd, t_min, chunk, fu, stream)
    if (B <= 4)
        CRSH_HIT(2);
    else if (B <= 8)
        CRSH_HIT(3);
    else if (B <= 16)
        CRSH_HIT(4);
    else
        CRSH_HIT(5);
#undef CRSH_HIT
}

uint32_t hit_pairs_launch(const hit_tris_ws &tri, const hit_slots_ws &hs,
                      const crsh_pairs *level1, int32_t bundle, const crsh_scene *scene, float t_min,
                      crsh_hits *hits, crsh_meta *meta, const batch_dev *bd, int32_t hit_block, hipStream_t stream,
                      bool packed, uint32_t tri_base)
{
    if (!level1->capacity) return 0u;
    const uint32_t chunk = (uint32_t)hit_block * (HIT_CHUNK / 256u);
    prof_scope ps("k_hit", stream);
    return packed ? k_hit_launch<HIT_PACKED>(hs, tri, level1, (uint32_t)bundle, hits, meta, scene->m, tri_base, bd,
                                             t_min, chunk, fused_in{}, stream)
                  : k_hit_launch<HIT_STORED>(hs, tri, level1, (uint32_t)bundle, hits, meta, scene->m, tri_base, bd,
                                             t_min, chunk, fused_in{}, stream);
}

// level-2 pairs with the pass bits of their children; `parts` workgroups of
// the launch before keep their counts.  rest: room for a word per HIT_TILE pairs,
// n_rest: a word that is zero.  Returns the workgroups that have counts.
uint32_t hit_masked_launch(const hit_tris_ws &tri, const hit_slots_ws &hs, const crsh_pairs *level2,
                           const uint32_t *mask, int32_t merge, int32_t bundle, const crsh_scene *scene, float t_min,
                           crsh_hits *hits, crsh_meta *meta, const batch_dev *bd, int32_t hit_block, uint32_t parts,
                           uint32_t *rest, uint32_t *n_rest, hipStream_t stream)
{
    uint32_t nf = 2;
    while (nf < (uint32_t)merge) nf *= 2;
    const uint32_t chunk = (uint32_t)hit_block * HIT_FUSED_PPT;
    fused_in fu{mask, nf, (uint32_t)merge, parts, rest, n_rest, false};
    prof_scope ps("k_hit", stream);
    if (nf <= 4)
        return std::max(parts, k_hit_launch<HIT_FUSED>(hs, tri, level2, (uint32_t)bundle, hits, meta, scene->m, 0u, bd,
                                                       t_min, chunk, fu, stream));
    for (int pass = 0; pass < 2; ++pass, fu.deferred = true)
        fu.parts = std::max(fu.parts, k_hit_launch<HIT_LISTED>(hs, tri, level2, (uint32_t)bundle, hits, meta, scene->m,
                                                               0u, bd, t_min, chunk, fu, stream));
    return fu.parts;
}

void hit_final_launch(const crsh_rays *sorted, const uint32_t *sorted_ids, const float4 *tri,
                      const hit_slots_ws &hs, int32_t bundle, const crsh_scene *scene, float t_min,
                      crsh_hits *hits, crsh_meta *meta, const batch_dev *bd, uint32_t n_part, hipStream_t stream)
{
    sorted_rays R{sorted->ox, sorted->oy, sorted->oz, sorted->dx, sorted->dy, sorted->dz, sorted->tmax};
    const batch_dev b = bd ? *bd : batch_dev{};
    uint32_t g = std::min<uint32_t>((sorted->capacity + 255) / 256, 4096);
    if (g == 0) g = 1;
    hit_out o{hits->tri, hits->t, hits->u, hits->v};
    prof_scope ps("k_hit_final", stream);
    if (bd)
        k_hit_final<true><<<g, 256, 0, stream>>>(R, tri, sorted_ids, t_min, hits->tkey, hs.keys, (uint32_t)bundle,
                                                 hs.slots, o, meta, sorted->capacity, scene->m, b, hs.part, n_part);
    else
        k_hit_final<false><<<g, 256, 0, stream>>>(R, tri, sorted_ids, t_min, hits->tkey, nullptr, (uint32_t)bundle,
                                                  0u, o, meta, sorted->capacity, scene->m, b, hs.part, n_part);
}

crsh_status hit_check(const crsh_rays *sorted, const uint32_t *sorted_ids, int32_t bundle, const crsh_pairs *level1,
                      const crsh_scene *scene, crsh_hits *hits, crsh_meta *meta, void *ws, int32_t hit_block,
                      const char *who)
{
    if (!sorted || !sorted_ids || !level1 || !scene || !hits || !meta || !ws) {
        set_error("%s: NULL argument", who);
        return CRSH_ERR_INVALID;
    }
    if (bundle < 1 || bundle > CRSH_MAX_BUNDLE) {
        set_error("%s: bundle must be in [1, %d]", who, CRSH_MAX_BUNDLE);
        return CRSH_ERR_INVALID;
    }
    if (hit_block != 64 && hit_block != 128 && hit_block != 256) {
        set_error("%s: workgroup size must be 64, 128 or 256", who);
        return CRSH_ERR_INVALID;
    }
    if (!sorted->ox || !sorted->oy || !sorted->oz || !sorted->dx || !sorted->dy || !sorted->dz ||
        !sorted->tmax || !hits->tkey || !hits->tri || !hits->t || !hits->u || !hits->v ||
        (level1->capacity && (!level1->tri || !level1->node))) {
        set_error("%s: incomplete arrays", who);
        return CRSH_ERR_INVALID;
    }
    for (int k = 0; k < 9; ++k)
        if (!scene->v[k] && scene->m) {
            set_error("%s: missing vertex array", who);
            return CRSH_ERR_INVALID;
        }
    if (hits->capacity < sorted->capacity) {
        set_error("%s: hit capacity below the ray capacity", who);
        return CRSH_ERR_INVALID;
    }
    // the final tests address ray slots (16 B in each of three arrays) and
    // triangles (48 B) by 32-bit byte offsets
    if ((uint64_t)sorted->capacity + (uint64_t)CRSH_MAX_FRAMES * (CRSH_MAX_BUNDLE - 1) > CRSH_HIT_MAX_SLOTS ||
        scene->m > CRSH_HIT_MAX_TRIS) {
        set_error("%s: at most %u ray slots and %u triangles", who, (unsigned)CRSH_HIT_MAX_SLOTS,
                  (unsigned)CRSH_HIT_MAX_TRIS);
        return CRSH_ERR_INVALID;
    }
    return CRSH_OK;
}

crsh_status hit_launch(const crsh_rays *sorted, const uint32_t *sorted_ids, int32_t bundle,
                       const crsh_pairs *level1, const crsh_scene *scene, float t_min, crsh_hits *hits,
                       crsh_meta *meta, void *ws, size_t ws_bytes, const batch_dev *bd, int32_t hit_block,
                       hipStream_t stream, bool packed, uint32_t tri_base)
{
    crsh_status st = hit_check(sorted, sorted_ids, bundle, level1, scene, hits, meta, ws, hit_block,
                               "crsh_closest_hit");
    if (st != CRSH_OK) return st;
    const uint32_t slots = hit_slots(sorted->capacity, bd != nullptr);
    if (ws_bytes < hit_ws_bytes(scene->m, slots)) {
        set_error("crsh_closest_hit: workspace too small (%zu < %zu)", ws_bytes, hit_ws_bytes(scene->m, slots));
        return CRSH_ERR_INVALID;
    }
    const hit_tris_ws tri = carve_hit_tris(ws, scene->m);
    const hit_slots_ws hs = carve_hit_slots((char *)ws + hit_tris_bytes(scene->m), slots);
    hit_pack_launch(scene, tri, sorted, hs, bundle, meta, bd, stream);
    const uint32_t parts = hit_pairs_launch(tri, hs, level1, bundle, scene, t_min, hits, meta, bd, hit_block, stream, packed,
                     tri_base);
    hit_final_launch(sorted, sorted_ids, tri.tri, hs, bundle, scene, t_min, hits, meta, bd, parts, stream);
    return hip_check(hipGetLastError(), "crsh_closest_hit launch");
}

}  // namespace crsh

extern "C" crsh_status crsh_closest_hit(const crsh_rays *sorted, const uint32_t *sorted_ids, int32_t bundle,
                                        const crsh_pairs *level1, const crsh_scene *scene, float t_min,
                                        crsh_hits *hits, crsh_meta *meta, void *ws, size_t ws_bytes,
                                        hipStream_t stream)
{
    return hit_launch(sorted, sorted_ids, bundle, level1, scene, t_min, hits, meta, ws, ws_bytes, nullptr, 256,
                      stream, false, 0u);
}

extern "C" crsh_status crsh_closest_hit_packed(const crsh_rays *sorted, const uint32_t *sorted_ids, int32_t bundle,
                                               const crsh_packed_pairs *level1, uint32_t tri_begin,
                                               const crsh_scene *scene, float t_min, crsh_hits *hits,
                                               crsh_meta *meta, void *ws, size_t ws_bytes, hipStream_t stream)
{
    if (!level1) {
        set_error("crsh_closest_hit_packed: NULL argument");
        return CRSH_ERR_INVALID;
    }
    if (level1->capacity && !level1->pair) {
        set_error("crsh_closest_hit_packed: incomplete arrays");
        return CRSH_ERR_INVALID;
    }
    // the packed words travel in the triangle array; no node array
    crsh_pairs p{level1->pair, level1->pair, level1->capacity};
    return hit_launch(sorted, sorted_ids, bundle, &p, scene, t_min, hits, meta, ws, ws_bytes, nullptr, 256, stream,
                      true, tri_begin);
}
