// Internal helpers shared by the host-side translation units of the library.
#pragma once

#include <stdint.h>

#include "lumo_tree.h"

namespace lumo {

// Record a printf-style message for lumo_last_error() and return `st`.
lumo_status fail(lumo_status st, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

// Seg record and seg_nodes entry widths of the plan blob.
constexpr int kSegWords = 4;      // {request, source cut, first entry, length}
constexpr int kSegNodeWords = 3;  // {absolute row, writes output, cut to export}
constexpr int kPreChunk = 32;     // preorder positions per chunk
constexpr int kPreStack = 16;     // path-stack candidate slots per chunk
constexpr int kPreCiWords = 4;    // candidate-slot words per preorder position (16 bytes)

// Preorder tables of WY plans whose paths have more than kPreStack + 1 nodes (and at most
// kDeepStack), behind the last named section of the blob: {mark, 0}, then per position the
// candidate slot of every ancestor (one byte per depth, kDeepStack bytes: m, or kDeepStack +
// its offset in the chunk; 0xff past the node's depth), then per chunk the rows of its path
// stack. Their offset, or -1 for a plan without them.
constexpr int kDeepStack = 32;
constexpr int kDeepHead = 2;
constexpr int32_t kDeepMark = 0xdeeb;
inline int64_t deep_words(const lumo_plan& p) {
    return kDeepHead + (int64_t)(kDeepStack / 4) * p.total_nodes + (int64_t)kDeepStack * p.n_chunks;
}
inline bool deep_plan(const lumo_plan& p) {
    return p.policy == LUMO_POLICY_WY && p.max_depth > kPreStack + 1 && p.max_depth <= kDeepStack;
}
inline int64_t deep_section(const lumo_plan& p, const int32_t* host_blob) {
    const int64_t at = p.o_vis + 2 * (int64_t)p.total_nodes;
    if (!deep_plan(p) || at + deep_words(p) > p.n_words) return -1;
    return host_blob[at] == kDeepMark ? at : -1;
}

// Traversal of the single-launch scan, behind the last named section of the blob of a
// sequential policy's plan: {slots, mark}, then {row, code} per node. Its offset, or -1 for a
// plan without it (the WY policy; words written before the section existed).
constexpr int kScanHead = 2;
constexpr int kScanWords = 2;
constexpr int32_t kScanMark = 0x5ca11;
inline int64_t scan_section(const lumo_plan& p, const int32_t* host_blob) {
    int64_t at = p.o_vis + 2 * (int64_t)p.total_nodes;
    at += at & 1;  // 8-byte entries
    if (p.policy == LUMO_POLICY_WY || at + kScanHead + kScanWords * (int64_t)p.total_nodes > p.n_words) return -1;
    return host_blob[at + 1] == kScanMark ? at : -1;
}

}  // namespace lumo
