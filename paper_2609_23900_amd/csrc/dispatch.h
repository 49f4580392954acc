// Host rules that choose between two forms of a kernel with the same results, from the plan
// and the dimensions alone.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "internal.h"

namespace lumo {

// Whether the single-launch scan (verify_scan.hip) is estimated to finish before the level-by-level
// one. It walks a tree's nodes one after the other, whatever their shape; the other form
// takes the longest segment of each level, and its launches, waves and cut states add up. Calls
// of more than 1,024 column tiles (four requests x 32 heads at d_v = 128) are bound by that
// work and always ran faster in the single launch. Below, the coefficients (microseconds;
// per launch, node of a longest segment, and thousand waves, node updates and cut tiles) are
// fitted to both forms over 236 calls of 1 to 32 requests, PATHS, TWO_LEVEL and
// RECOMPUTE, d_k = 16 to 128: 64-node trees to stars of 256 nodes. The choice is at most 5%
// behind the better form in each. One request, one layer, 32 heads, d = 128: 256 leaves under a
// root 48 us by level, 143 us in one launch; 256 nodes of 8 levels, TWO_LEVEL 109 and 143
// us, PATHS 178 and 143 us; 64 nodes of 8 levels, PATHS 99 and 39 us.
inline bool scan_tree_faster(const lumo_gdn_dims& d, const lumo_plan& p, const int32_t* host_blob) {
    if ((int64_t)d.n_req * d.n_layers * d.h_v * (d.d_v / 16) > 1024) return true;
    const float s = (float)d.d_k / 128.f;
    const float kilo = (float)(d.n_layers * d.h_v * ((d.d_v + 63) / 64)) * 1e-3f;  // waves per segment
    const float node = d.d_k == 128 ? 0.56f : d.d_k == 64 ? 0.37f : d.d_k == 32 ? 0.48f : 0.21f;
    const float tree = 4.f + node * (float)p.max_nodes;
    float level = (2.5f + 5.f * s) * (float)p.n_levels + kilo * (0.9f * s * (float)p.n_seg + (0.06f + 0.7f * s) * (float)p.n_seg_nodes +
                                                                 5.f * s * (float)p.n_cuts);
    const float step = 0.4f + 1.6f * s;
    if (level + step * (float)p.max_seg_len >= tree) return true;
    for (int lv = 0; lv < p.n_levels; ++lv) {
        int longest = 0;
        for (int i = host_blob[p.o_level_off + lv]; i < host_blob[p.o_level_off + lv + 1]; ++i)
            longest = std::max(longest, (int)host_blob[p.o_seg + kSegWords * (int64_t)i + 3]);
        level += step * (float)longest;
    }
    return level >= tree;
}

}  // namespace lumo
