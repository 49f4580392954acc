// Host rules that choose between two forms of a kernel with the same results, from the plan
// and the dimensions alone.
#pragma once

#include <stdint.h>

#include <algorithm>

#include "internal.h"

namespace lumo {

// Whether the single-launch scan (verify_scan.hip) is estimated to finish before the level-by-level
// one. It walks a tree's nodes one after the other, whatever their shape; the other form
// takes the longest segment of each level, and its launches, waves and cut states add up. Both
// estimates in microseconds, linear in the plan: a node walked or a step of a longest segment,
// and per thousand column tiles (16 columns there, 64 here) a request's or segment's state, a node
// and a cut state. Coefficients are fitted per key length to both forms, apart for calls of
// more and of less than 1,024 16-column tiles (the device full or not), over 7,575 calls of 1
// to 64 requests, chains, stars and trees of 2 to 20 levels with 1 to 256 nodes under PATHS,
// TWO_LEVEL and RECOMPUTE. Of these the choice is more than 5% behind the better form in 48 (at
// most 32%), and more than 5% behind the level-by-level form in 29. One layer, 32 heads, d = 128,
// level by level and in one launch: one request, 256 leaves under a root 48 and 143 us; 256
// nodes of 8 levels, TWO_LEVEL 109 and 143 us, PATHS 178 and 143 us; 64 nodes of 8 levels,
// PATHS 99 and 39 us; 64 requests of one node 24 and 32 us, of 8 in a chain 67 and 58 us.
struct ScanCost {
    float tree, tree_node, tree_state, tree_work;                // single launch
    float level, level_step, level_state, level_work, level_cut;  // level by level
};
inline bool scan_tree_faster(const lumo_gdn_dims& d, const lumo_plan& p, const int32_t* host_blob) {
    // key lengths of 16, 32, 64 and 128
    static const ScanCost small[4] = {{2.374f, 0.236f, 1.432f, 0.085f, 2.275f, 0.645f, 0.641f, 0.061f, 0.736f},
                                      {3.260f, 0.470f, 0.013f, 0.012f, 2.678f, 0.815f, 0.108f, 0.232f, 1.834f},
                                      {3.333f, 0.338f, 0.245f, 0.021f, 3.231f, 0.935f, 0.242f, 0.389f, 11.231f},
                                      {4.712f, 0.463f, 0.684f, 0.025f, 4.422f, 1.639f, 0.529f, 0.763f, 20.296f}};
    static const ScanCost large[4] = {{1.801f, 0.191f, 0.913f, 0.031f, 1.734f, 0.705f, 0.210f, 0.219f, 1.223f},
                                      {3.736f, 0.525f, 0.558f, 0.037f, 1.567f, 0.946f, 0.481f, 0.262f, 2.235f},
                                      {1.884f, 0.196f, 1.142f, 0.089f, 2.340f, 1.010f, 0.332f, 0.720f, 5.153f},
                                      {2.107f, 0.286f, 1.658f, 0.194f, 2.461f, 2.576f, 1.058f, 1.278f, 8.610f}};
    const float heads = (float)d.n_layers * (float)d.h_v * 1e-3f;
    const float narrow = heads * (float)(d.d_v / 16), wide = heads * (float)((d.d_v + 63) / 64);
    const int key = d.d_k == 16 ? 0 : d.d_k == 32 ? 1 : d.d_k == 64 ? 2 : 3;
    const ScanCost& c = (narrow * (float)d.n_req > 1.024f ? large : small)[key];
    const float tree = c.tree + c.tree_node * (float)p.max_nodes +
                       narrow * (c.tree_state * (float)d.n_req + c.tree_work * (float)p.total_nodes);
    float level = c.level * (float)p.n_levels + wide * (c.level_state * (float)p.n_seg + c.level_work * (float)p.n_seg_nodes +
                                                        c.level_cut * (float)p.n_cuts);
    if (level + c.level_step * (float)p.max_seg_len >= tree) return true;
    for (int lv = 0; lv < p.n_levels; ++lv) {
        int longest = 0;
        for (int i = host_blob[p.o_level_off + lv]; i < host_blob[p.o_level_off + lv + 1]; ++i)
            longest = std::max(longest, (int)host_blob[p.o_seg + kSegWords * (int64_t)i + 3]);
        level += c.level_step * (float)longest;
    }
    return level >= tree;
}

// Whether the WY form on the vector ALUs (verify_wyv.hip) is estimated to finish before the
// matrix-core one, where both serve the plan: fp32 operands, and bf16 with paths of more than 17
// nodes, at d = 128. The matrix-core kernels pay for whole chunks and half-chunks (16
// nodes), the vector one node by node, so tiny trees are its own. Estimated are the work of all
// heads and the largest tree's serial time; they overlap to four fifths with trees of one
// size and hardly where one large tree is left at the end. Coefficients in microseconds, from
// trees of 1 to 66 nodes, 8 to 8,192 heads. Matrix cores (vector ALUs): one node 32 heads 10.0
// (5.4), 2,048 heads 47 (24); four nodes 32 heads 10.0 (11.5), 2,048 heads 47 (37); 9 nodes 47
// (61). Chains of 18, 2,048 heads, 143 (117), of 24 134 (151). 8,192 heads, 63 requests of one
// node beside one of 18: 363 (136), bf16 171 (137), beside one of 64 in 8 levels 194 (242).
inline bool wy_vector_faster(const lumo_gdn_dims& d, const lumo_plan& p, const int32_t* host_blob) {
    const bool f32 = d.op_dtype == LUMO_F32, deep = p.max_depth > kPreStack + 1;
    if (!f32 && !deep) return false;
    const float chunk = !f32 ? 0.0104f : deep ? 0.0235f : p.max_depth > 9 ? 0.02f : 0.0127f;  // a request's first
    const float half = !f32 ? 0.0105f : deep ? 0.0215f : 0.01f;
    const float depth = (float)p.max_depth;
    int64_t requests = 0, halves = 0;
    for (int r = 0; r < d.n_req; ++r) {
        const int n = host_blob[p.o_node_off + r + 1] - host_blob[p.o_node_off + r];
        requests += n > 0;
        halves += (n + kPreChunk / 2 - 1) / (kPreChunk / 2);
    }
    const float apart = 0.8f - 0.6f * (float)p.total_nodes / (float)std::max<int64_t>(1, requests * p.max_nodes);
    auto time = [&](float work, float serial) { return std::max(work, serial) + apart * std::min(work, serial); };
    const float heads = (float)d.n_layers * (float)d.h_v;
    const float vector = time(heads * (0.0085f * (float)requests + (0.0022f + 3e-5f * depth) * (float)p.total_nodes),
                              3.f + (float)p.max_nodes * (2.1f + 0.025f * depth));
    const float matrix = time(heads * (chunk * (float)requests + 0.01f * (float)(p.n_chunks - requests) + half * (float)halves),
                              (deep ? 17.f : p.max_depth > 9 ? 12.f : 10.f) +
                                  8.5f * (float)((p.max_nodes + kPreChunk - 1) / kPreChunk - 1));
    return vector < matrix;
}

// Whether the commit's replay (commit.hip) takes wavefronts of 16 value columns rather than 64.
// Both are bound by the state bank's way through HBM or the Infinity Cache; 16 columns keep
// more of it in flight and shorten each path step, 64 read whole rows and share each key row.
// So 16 while the bank stays in the 256 MB cache between calls, and for heads that leave
// columns of a 64-wide tile idle (d = 128 x 16, 768 heads, 8 steps: 20.0 -> 10.0 us); with d_k =
// 128 at every such size (8 steps, bf16: 32 heads 18.5 -> 10.0, 512 25.3 -> 20.5, 3,072
// 86.4 -> 72.8 us), with shorter keys, whose steps are short already, up to 1,024 tiles of 64
// columns, one wave per SIMD, and 1,536 in bf16 (bf16 d = 64 x 128, 8 steps: 512 heads 16.5 ->
// 14.2 us, 768 18.3 -> 17.7, 2,048 33.0 -> 39.4; fp32 d = 32 x 128: 256 heads 9.4 -> 8.3 us, 768 11.7
// -> 12.3, 2,048 21.6 -> 26.0, 12,288 88 -> 109). Steps are few where the trees or max_path are
// short: up to three steps, 512 of these tiles (bf16, d = 128 x 128, 512 heads: one step 14.3
// against 17.2 us, two 1.12 times, four as long), except where a step converts nothing
// (fp32, d_k = 128: 0.89 to 1.04 times).
// Beyond 256 MB: bf16, d = 128, 18 layers x 8 requests x 32 heads 122 against 136 us.
inline bool replay_narrow(const lumo_gdn_dims& d, const lumo_plan& p, int max_path) {
    const int64_t heads = (int64_t)d.n_req * d.n_layers * d.h_v;
    const int64_t tiles = heads * ((d.d_v + 63) / 64);
    if (heads * d.d_k * d.d_v * (int64_t)sizeof(float) > (int64_t(256) << 20)) return false;
    const bool few = std::min(max_path, (int)p.max_depth) <= 3;
    if (d.d_v <= 32) return !few || d.d_k > 32 || tiles <= 1024;
    if (d.d_k == 128) return !few || d.op_dtype == LUMO_F32 || tiles <= 512;
    return tiles <= (few ? 512 : d.op_dtype == LUMO_F32 ? 1024 : 1536);
}

// The conv's walk over runs (conv.hip): nodes per run and channels per lane, 0 nodes where the
// run kernel is faster. A run starts by loading its ancestors and weights, and the grid has
// as many runs for every request as the largest one needs. So the walk takes calls
//  - of at least 2,048 blocks' work (eight one-wave blocks per CU), with root paths that
//    leave LDS for eight blocks per CU (20 KB);
//  - whose runs, where a request has several, are mostly full: six tenths in fp32 (32 requests x
//    33 nodes, 4 layers x 8,192 channels: run kernel 84, walk 63 us; 128 requests x 17 nodes, 2
//    layers: 88 and 99 us), three quarters in bf16 (32 x 96 nodes, 4 layers: 111 and 113
//    us; 64 x 65 nodes, 2 layers: 77 and 96 us);
//  - with enough of the blocks in use: a fifth in fp32, where they are short (256 and 31 x 32
//    nodes, 2 layers x 8,192 channels: 35 and 48 us), half in bf16 (4 requests x 512 and 28 x
//    64 nodes, 4 layers x 8,192: 135 and 232 us; 16 requests of 256 and 32 nodes in turn: 92
//    and 95 us);
//  - whose work is spread over the XCDs, each of which takes an eighth of the layers' requests in
//    order: the busiest at most 1.5 times the average (4 requests x 512 and 28 x 64 nodes, fp32, 1
//    layer x 8,192: 4.3 times, 48 and 131 us; 4 layers: 1.47 times, 303 and 298 us; 6
//    layers x 2,304: 168 and 112 us. Dealt over the XCDs instead, requests of 256 and 32
//    nodes in turn took 1.4 times as long).
// fp32 operands take runs of 16 nodes: 8 requests x 12 layers x 64 nodes x 8,192 channels 125 ->
// 82 us, 3 layers 22.9 -> 18.2 us; below the line 11.8 against 11.3 us, paths of 32 nodes 22.9
// against 26.9. bf16 rows are half as long, so a run has to be longer to pay for its start:
// 64 nodes (32 requests x 256 nodes 69 -> 57 us).
struct ConvWalk {
    int run_nodes, lane_channels;
};
inline ConvWalk conv_walk(const lumo_gdn_dims& d, const lumo_plan& p, const int32_t* host_blob, int channels) {
    const bool bf = d.op_dtype == LUMO_BF16;
    const ConvWalk walk{bf ? 64 : 16, bf ? 8 : 4}, none{0, 0};
    const int64_t chunks = (channels + 64 * walk.lane_channels - 1) / (64 * walk.lane_channels);
    if (p.max_depth + 3 > 20 || (int64_t)p.total_nodes / walk.run_nodes * d.n_layers * chunks < 2048) return none;
    const int64_t most = (p.max_nodes + walk.run_nodes - 1) / walk.run_nodes;
    int64_t runs = 0;
    for (int r = 0; r < d.n_req; ++r) {
        const int n = host_blob[p.o_node_off + r + 1] - host_blob[p.o_node_off + r];
        runs += (n + walk.run_nodes - 1) / walk.run_nodes;
    }
    if (most > 1 && 20 * (int64_t)p.total_nodes < (bf ? 15 : 12) * walk.run_nodes * runs) return none;
    if ((bf ? 2 : 5) * runs < d.n_req * most) return none;
    // nodes of the layers' requests before position x / 8
    const int64_t total = p.total_nodes;
    auto before = [&](int64_t x) {
        const int64_t i = x / 8, r = i % d.n_req;
        const int32_t* off = host_blob + p.o_node_off + r;
        return 8 * (i / d.n_req * total + off[0]) + x % 8 * (int64_t)(off[1] - off[0]);
    };
    const int64_t per = (int64_t)d.n_req * d.n_layers;
    for (int k = 0; k < 8; ++k)
        if (2 * (before((k + 1) * per) - before(k * per)) > 3 * d.n_layers * total) return none;
    return walk;
}

}  // namespace lumo
