// Device types and launchers of the traversal shared with the fused last
// level (crsh_leaf_hit).
#pragma once

#include "batch.hpp"

namespace crsh {

// One level's pairs: two arrays (triangle, node), or one packed word per
// pair -- node in the high bits, triangle minus tri_base in the low
// CRSH_PACKED_TRI_BITS (Sec. 3.3.7's 32-bit pair encoding; node == nullptr).
struct pairs_dev {
    uint32_t *tri, *node;
    uint64_t cap;
    uint32_t packed;       // 1: packed words in `tri`
    uint32_t tri_base;     // first triangle of the batch (packed form)
};

// PACKED is a compile-time choice so that the two-array kernels are the
// same code as without packed support.
template <bool PACKED>
__device__ __forceinline__ void pair_put(const pairs_dev &p, uint64_t at, uint32_t tri, uint32_t node)
{
    if constexpr (PACKED) {
        p.tri[at] = (node << CRSH_PACKED_TRI_BITS) | (tri - p.tri_base);
    } else {
        p.tri[at] = tri;
        p.node[at] = node;
    }
}

struct pair_levels {
    pairs_dev p[CRSH_MAX_LEVELS];
};
struct node_arrays {
    const float *cx, *cy, *cz, *r, *ax, *ay, *az, *c, *tan, *sec;
};

// per-level scratch carved from the workspace
struct trav_scratch {
    uint64_t top_cap;      // entries of cnt_top
    uint32_t top_many;     // most parts per top-level item where there are many items
    uint32_t *cnt_top;     // survivors per top-level item
    uint32_t *cnt;         // surviving children per tile of pairs (cleared by the scan that reads it)
    uint64_t *off;         // exclusive offsets of the items or tiles
    void *mask[2];         // pass bits of a level's pairs, by the parity of the level
    uint32_t *bits;        // pass masks of the fused last level's count pass
    uint64_t *scan_flags;  // look-back words of the scan
    uint32_t n_flags;
    uint32_t *scan_ctr;    // tile counter of the scan
    uint64_t *part;        // node tests per workgroup (TRAV_PARTS, cleared by the scan that adds them up)
    uint64_t *top_part;    // three counts per workgroup of the top-level count
};

constexpr uint32_t SCAN_THREADS = 1024;
constexpr uint32_t SCAN_ITEMS = 4;
constexpr uint32_t SCAN_GRID = 128;        // most blocks of a scan
constexpr uint32_t SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;
static_assert(SCAN_TILE == SCAN_TILE_ITEMS, "workspace sizing");

// spheres of the triangles [tri_begin, tri_end), packed nodes; n_cnt survivor
// counts of S.cnt cleared (0: S left alone), levels: see k_trav_prep
void trav_prep_launch(const crsh_scene *scene, uint32_t tri_begin, uint32_t tri_end, float4 *tsph,
                      const crsh_nodes *nodes, crsh_meta *meta, float4 *na, float4 *nb, float *ns,
                      const trav_scratch &S, uint64_t n_cnt, uint32_t levels, hipStream_t stream);
// count pass of one level (pass masks and per-tile survivor counts in S,
// node tests added to meta)
void level_count_launch(int32_t parent_level, int32_t merge, const float4 *na, const float4 *nb, const float *ns,
                        const float4 *tsph, uint32_t m, const pair_levels &P, const trav_scratch &S, crsh_meta *meta,
                        const batch_dev *bd, uint64_t tiles_cap, uint32_t top_levels, hipStream_t stream);

}  // namespace crsh
