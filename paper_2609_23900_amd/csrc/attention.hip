// Tree attention on the matrix cores (Sec. V-B; visibility Sec. III-A).
//
// A query row is (tree node, query head); it sees its request's committed context and the
// tree nodes on its own root-to-node path. Split-K, as in flash-decoding: the key tiles of
// a (request, key/value head) -- the context's 64-key tiles, then the tree's own -- are cut
// into contiguous ranges; a block serves one range for a chunk of query rows, taken from
// all the nodes and all the query heads that share the key/value head, so every staged key
// and value tile is used by all of them. A second kernel merges the ranges through their
// log-sum-exp; with one range the block writes the result itself.
//
// A wavefront holds R tiles of 16 query rows (R = 1, 2), one row per lane column. Every
// key and value fragment read from LDS feeds R matrix instructions: at R = 1 the LDS port
// (128 B per clock for four SIMDs) needs twice the time of the matrix cores, at R = 2 as
// much as they do, so calls with many rows per key/value head (compute-bound) take R = 2;
// calls of up to 64 rows are bound by HBM and take R = 1 (rule in attn_shape).
//
// Layout per wavefront. The scores are computed transposed, S^T = K Q^T (16x16x32 bf16
// MFMA), so that a lane holds 16 scores of ONE query row per tile (4 lane groups split
// the 64 keys): the running maximum needs two lane-group swaps per tile, the sum only
// one reduction at the end, and the probabilities are already in the B-operand layout of
// O^T = V^T P^T (key slot 8 j + e of lane group j is key 4 j + e of the tile's first
// 16-key half for e < 4, of the second for e >= 4). K and V tiles are staged by direct
// global-to-LDS copies, key-major, 16-byte slot c of key t at position c ^ swz(t), with
// swz a rotation of t's low four bits: the 16 keys of a K fragment read take 16 different
// slots, and the four keys of a transposing V read (ds_read_b64_tr_b16: within 16 lanes,
// lane i receives element i % 4 of lanes 4 e + i / 4, e = 0..3) four different slot pairs.
// The probabilities of a tile are taken relative to the row's largest score in that tile, so
// that its largest is exactly 1 when they are rounded to bf16, and the tile's product is added
// to the output with its weight relative to the running maximum: the rounding is that of
// one range per tile, however long the ranges are. Relative to the running maximum
// itself, 8 requests of 64 nodes x 32 heads over 16,384 tokens had an error of 2.26e-3 against
// 64 bits instead of 2.09e-3 (bf16 outputs alone 1.7e-3), in 147 us instead of 156 us.
// Tiles of 64 keys, double-buffered. Visibility inside the tree comes from the plan's
// preorder intervals; only ragged context tiles and tree tiles are masked.
#include <algorithm>
#include <mutex>

#include "device_common.h"
#include "internal.h"
#include "launch.h"

namespace lumo {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void lds_void;
typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

constexpr int kAD = 128;  // head dimension
constexpr int kAT = 64;   // keys per tile
constexpr int kAW = 4;    // wavefronts per block

struct AttnParams {
    const int32_t* blob;
    int32_t o_node_off, o_row_off, o_vis;
    const int32_t* ctx_off;
    int32_t n_req, h_q, h_kv, n_range, n_chunk, total_rows, max_nodes;
    int32_t xcd_unit;    // blocks dealt to an XCD together
    int32_t group_log2;  // log2 of the query heads per key/value head
    float scale_log2;    // scale * log2(e): scores in the base-2 domain
    const uint16_t* q;
    const uint16_t* k_ctx;
    const uint16_t* v_ctx;
    const uint16_t* k_tree;
    const uint16_t* v_tree;
    float* ws_o;    // [n_range][total_rows][h_q][kAD]: normalised partial outputs
    float* ws_lse;  // [n_range][total_rows][h_q]: partial log2-sum-exp2 (-inf: no key)
    uint16_t* o;    // [total_rows][h_q][kAD]
    float* lse;     // [total_rows][h_q]
};

// max / sum over the four 16-lane rows (the same in every lane)
__device__ __forceinline__ float rows_max(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows_sum(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 w) { return __builtin_bit_cast(bf16x8, w); }

// a node's preorder position and the end of its subtree (4-byte aligned in the blob)
struct Interval {
    int x, y;
};

// position of key t's 16-byte slots: t's low four bits rotated left by one
__device__ __forceinline__ int swz(int t) { return ((t << 1) & 14) | ((t >> 3) & 1); }

// Two blocks of four waves per CU (64 KB of LDS, at most 256 registers each).
template <int R>
__global__ __launch_bounds__(64 * kAW, 2) void attn_kernel(AttnParams p) {
    constexpr int nthr = 64 * kAW;
    constexpr int kRows = 16 * R * kAW;  // query rows per block
    // key and value tiles: [key][16 slots]; slot c of key t holds dims 8 (c ^ swz(t)) .. + 7
    __shared__ uint4 kt0[kAT * 16];
    __shared__ uint4 kt1[kAT * 16];
    __shared__ uint4 vt0[kAT * 16];
    __shared__ uint4 vt1[kAT * 16];
    const int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int lq = lane & 15, lg = lane >> 4;

    // the row chunks of one key range run next to each other on one XCD, whose L2 serves
    // the range's keys and values to all of them; the units (launch_parts) go round-robin
    // over the XCDs, so that requests of different context lengths spread over all of them
    int blk = xcd_units(blockIdx.x, gridDim.x, p.xcd_unit);
    const int nc = blk % p.n_chunk;
    blk /= p.n_chunk;
    const int sp = blk % p.n_range;
    blk /= p.n_range;
    const int g = blk % p.h_kv;
    const int r = blk / p.h_kv;
    const int base = p.blob[p.o_node_off + r];
    const int N = p.blob[p.o_node_off + r + 1] - base;
    const int M = N << p.group_log2;  // query rows of this key/value head: row m is node
                                      // m >> group_log2, head m & (group - 1)
    if (kRows * nc >= M) return;  // uniform: no query row in this chunk
    const int rbase = p.blob[p.o_row_off + r];
    // this range's tiles [i0, i1) of the context's nct tiles and the tree's behind them
    const int c0 = p.ctx_off[r];
    const int nk = p.ctx_off[r + 1] - c0;
    const int nct = (nk + kAT - 1) / kAT;
    const int nt = nct + (N + kAT - 1) / kAT;
    const int per = (nt + p.n_range - 1) / p.n_range;
    const int i0 = sp * per, i1 = min(nt, i0 + per);

    const int m0 = kRows * nc + 16 * R * wave;  // uniform: the wave's first row
    const bool wact = m0 < M;                   // uniform: idle waves only copy tiles
    int slot[R], head[R];
    uint4 qf[R][kAD / 32];  // B operands: dims 32 ks + 8 (lane / 16) .. + 7 of the lane's row
#pragma unroll
    for (int t = 0; t < R; ++t) {
        const int m = min(m0 + 16 * t + lq, M - 1);
        slot[t] = m >> p.group_log2;
        head[t] = (g << p.group_log2) + (m & ((1 << p.group_log2) - 1));
#pragma unroll
        for (int ks = 0; ks < kAD / 32; ++ks)
            qf[t][ks] = *reinterpret_cast<const uint4*>(p.q + ((long)(rbase + slot[t]) * p.h_q + head[t]) * kAD +
                                                        32 * ks + 8 * lg);
    }

    // tile i into K and V buffers: keys past the end repeat the last key (masked later, so
    // pad rows and other requests' tokens are never read)
    auto tile_issue = [&](int i, uint4* kd, uint4* vd) {
        const bool tree = i >= nct;
        const uint16_t* km = tree ? p.k_tree : p.k_ctx;
        const uint16_t* vm = tree ? p.v_tree : p.v_ctx;
        const int row0 = tree ? rbase : c0;
        const int last = (tree ? N : nk) - 1;
        const int lo = (tree ? i - nct : i) * kAT;
#pragma unroll
        for (int j = 0; j < kAT * 16 / nthr; ++j) {
            const int slot0 = j * nthr + 64 * wave;  // uniform
            const int t = (slot0 + lane) >> 4;
            const int kb = (lane & 15) ^ swz(t);
            const long at = ((long)(row0 + min(lo + t, last)) * p.h_kv + g) * kAD + 8 * kb;
            __builtin_amdgcn_global_load_lds(km + at, (lds_void*)&kd[slot0], 16, 0, 0);
            __builtin_amdgcn_global_load_lds(vm + at, (lds_void*)&vd[slot0], 16, 0, 0);
        }
    };

    float mx[R], lsum[R];  // running max (base 2) of the rows, the lane's part of their sums
    f32x4 o[R][kAD / 16];
#pragma unroll
    for (int t = 0; t < R; ++t) {
        mx[t] = -1e30f;
        lsum[t] = 0.f;
#pragma unroll
        for (int dt = 0; dt < kAD / 16; ++dt)
#pragma unroll
            for (int x = 0; x < 4; ++x) o[t][dt][x] = 0.f;
    }

    auto compute = [&](int i, const uint4* kt, const uint4* vt) {
        // S^T = K Q^T: lane (row lane%16) gets keys 16 tt + 4 (lane/16) + x
        f32x4 s[R][kAT / 16];
#pragma unroll
        for (int tt = 0; tt < kAT / 16; ++tt) {
#pragma unroll
            for (int t = 0; t < R; ++t)
#pragma unroll
                for (int x = 0; x < 4; ++x) s[t][tt][x] = 0.f;
            const int key = 16 * tt + lq;
#pragma unroll
            for (int ks = 0; ks < kAD / 32; ++ks) {
                const bf16x8 a = as_bf16x8(kt[key * 16 + ((4 * ks + lg) ^ swz(key))]);
#pragma unroll
                for (int t = 0; t < R; ++t)
                    s[t][tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, as_bf16x8(qf[t][ks]), s[t][tt], 0, 0, 0);
            }
        }
        // masks (uniform branches): a ragged context tile's keys past the end, and the
        // tree keys whose subtree does not hold the row's node
        if (i < nct) {
            const int n = nk - i * kAT;
            if (n < kAT) {
#pragma unroll
                for (int t = 0; t < R; ++t)
#pragma unroll
                    for (int tt = 0; tt < kAT / 16; ++tt)
#pragma unroll
                        for (int x = 0; x < 4; ++x)
                            if (16 * tt + 4 * lg + x >= n) s[t][tt][x] = -INFINITY;
            }
        } else {
            const int lo = (i - nct) * kAT;
            const Interval* vis = reinterpret_cast<const Interval*>(p.blob + p.o_vis) + base;
            int pos[R];
#pragma unroll
            for (int t = 0; t < R; ++t) pos[t] = vis[slot[t]].x;
#pragma unroll
            for (int tt = 0; tt < kAT / 16; ++tt)
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const int sl = lo + 16 * tt + 4 * lg + x;
                    const Interval iv = vis[min(sl, N - 1)];
#pragma unroll
                    for (int t = 0; t < R; ++t)
                        if (sl >= N || pos[t] < iv.x || pos[t] >= iv.y) s[t][tt][x] = -INFINITY;
                }
        }
        // the tile's probabilities relative to the row's largest score in the tile (never above
        // 1), and the weight w of the tile relative to the running maximum
        float w[R];
#pragma unroll
        for (int t = 0; t < R; ++t) {
            float mt = fmaxf(fmaxf(s[t][0][0], s[t][0][1]), fmaxf(s[t][0][2], s[t][0][3]));
#pragma unroll
            for (int tt = 1; tt < kAT / 16; ++tt)
                mt = fmaxf(mt, fmaxf(fmaxf(s[t][tt][0], s[t][tt][1]), fmaxf(s[t][tt][2], s[t][tt][3])));
            mt = fmaxf(rows_max(mt) * p.scale_log2, -1e30f);  // finite also where no key is visible
            const float mn = fmaxf(mx[t], mt);
            if (__any(mn > mx[t])) {  // uniform; otherwise the factor is exactly 1
                const float corr = __builtin_amdgcn_exp2f(mx[t] - mn);
                mx[t] = mn;
                lsum[t] *= corr;
#pragma unroll
                for (int dt = 0; dt < kAD / 16; ++dt)
#pragma unroll
                    for (int x = 0; x < 4; ++x) o[t][dt][x] *= corr;
            }
            w[t] = __builtin_amdgcn_exp2f(mt - mn);
            float ls = 0.f;
#pragma unroll
            for (int tt = 0; tt < kAT / 16; ++tt)
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    s[t][tt][x] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][tt][x], p.scale_log2, -mt));
                    ls += s[t][tt][x];
                }
            lsum[t] = __builtin_fmaf(w[t], ls, lsum[t]);
        }
        bf16x8 pw[2][R];  // the two 32-key halves
#pragma unroll
        for (int kh = 0; kh < 2; ++kh)
#pragma unroll
            for (int t = 0; t < R; ++t)
                pw[kh][t] = as_bf16x8(make_uint4(f32x2_to_bf16x2(s[t][2 * kh][0], s[t][2 * kh][1]),
                                                 f32x2_to_bf16x2(s[t][2 * kh][2], s[t][2 * kh][3]),
                                                 f32x2_to_bf16x2(s[t][2 * kh + 1][0], s[t][2 * kh + 1][1]),
                                                 f32x2_to_bf16x2(s[t][2 * kh + 1][2], s[t][2 * kh + 1][3])));
        // O^T += w V^T P^T. Transposing reads: lane j of a 16-lane group reads dims 16 dt + 4 (j
        // % 4) .. + 3 of key 32 kh + 4 (lane / 16) + j / 4 (and of that key + 16), and receives
        // dim 16 dt + j of keys 32 kh + 4 (lane / 16) + e (and + 16 + e), e = 0..3
        const char* vb = reinterpret_cast<const char*>(vt);
#pragma unroll
        for (int dt = 0; dt < kAD / 16; ++dt) {
            const int sg = 2 * dt + ((lq & 3) >> 1);  // 16-byte dim segment, then its half
            const int hb = 8 * (lq & 1);
            f32x4 acc[R];
#pragma unroll
            for (int t = 0; t < R; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kh = 0; kh < 2; ++kh) {
                const int t1 = 32 * kh + 4 * lg + (lq >> 2), t2 = t1 + 16;
                const v4i16 r1 =
                    __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(vb + (t1 * 16 + (sg ^ swz(t1))) * 16 + hb));
                const v4i16 r2 =
                    __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(vb + (t2 * 16 + (sg ^ swz(t2))) * 16 + hb));
                const uint2 a1 = __builtin_bit_cast(uint2, r1), a2 = __builtin_bit_cast(uint2, r2);
                const bf16x8 va = as_bf16x8(make_uint4(a1.x, a1.y, a2.x, a2.y));
#pragma unroll
                for (int t = 0; t < R; ++t)
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pw[kh][t], acc[t], 0, 0, 0);
            }
#pragma unroll
            for (int t = 0; t < R; ++t)
#pragma unroll
                for (int x = 0; x < 4; ++x) o[t][dt][x] = __builtin_fmaf(w[t], acc[t][x], o[t][dt][x]);
        }
    };

    if (i0 < i1) {
        // copies of a tile have landed for every wave, and every wave is done with the
        // buffers that the next copies overwrite
        auto landed = [&]() {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        };
        tile_issue(i0, kt0, vt0);
        landed();
        for (int i = i0; i < i1; i += 2) {
            // tile i from buffers 0 while tile i + 1 lands in buffers 1, then the reverse
            const bool n1 = i + 1 < i1;
            if (n1) tile_issue(i + 1, kt1, vt1);
            if (wact) compute(i, kt0, vt0);
            if (!n1) break;
            landed();
            const bool n2 = i + 2 < i1;
            if (n2) tile_issue(i + 2, kt0, vt0);
            if (wact) compute(i + 1, kt1, vt1);
            if (!n2) break;
            landed();
        }
    }
    if (!wact) return;
    // normalised (partial) output and its log-sum-exp (-inf when no key was visible)
#pragma unroll
    for (int t = 0; t < R; ++t) lsum[t] = rows_sum(lsum[t]);
#pragma unroll
    for (int t = 0; t < R; ++t) {
        const float ls = lsum[t];
        if (m0 + 16 * t + lq >= M) continue;
        const float l2 = ls != 0.f ? mx[t] + __log2f(ls) : -INFINITY;  // NaN scores stay NaN
        const long ri = (long)(rbase + slot[t]) * p.h_q + head[t];
        if (p.n_range == 1) {  // uniform: nothing to merge
            const float inv = 1.f / ls;
#pragma unroll
            for (int dt = 0; dt < kAD / 16; ++dt)
                *reinterpret_cast<uint2*>(p.o + ri * kAD + 16 * dt + 4 * lg) =
                    make_uint2(f32x2_to_bf16x2(o[t][dt][0] * inv, o[t][dt][1] * inv),
                               f32x2_to_bf16x2(o[t][dt][2] * inv, o[t][dt][3] * inv));
            if (lane < 16) p.lse[ri] = l2 * 0.69314718055994531f;
            continue;
        }
        const long wi = (long)sp * p.total_rows * p.h_q + ri;
        const float inv = ls != 0.f ? 1.f / ls : 0.f;
#pragma unroll
        for (int dt = 0; dt < kAD / 16; ++dt)
            *reinterpret_cast<float4*>(p.ws_o + wi * kAD + 16 * dt + 4 * lg) =
                make_float4(o[t][dt][0] * inv, o[t][dt][1] * inv, o[t][dt][2] * inv, o[t][dt][3] * inv);
        if (lane < 16) p.ws_lse[wi] = l2;
    }
}

// Merge of the key ranges of one (query row, head): weights 2^(lse_s - max), each lane two
// of the d values, eight ranges' loads in flight, a fixed summation order, so the result
// does not depend on timing. KW waves per (row, head): four take every fourth range each
// and their sums are added in order (many ranges: one long context; few pairs); one (few
// ranges, many rows) leaves a block of four waves four (row, head) pairs.
template <int KW>
__global__ __launch_bounds__(256) void attn_combine_kernel(AttnParams p) {
    __shared__ float red[4];
    __shared__ float2 part[4][64];
    const int t = (int)threadIdx.x, lane = t & 63, wv = t >> 6;
    long blk = KW == 4 ? (long)blockIdx.x : 4 * (long)blockIdx.x + wv;
    const int h = (int)(blk % p.h_q);
    blk /= p.h_q;
    const int s = (int)(blk % p.max_nodes);
    const int r = (int)(blk / p.max_nodes);
    if (r >= p.n_req) return;  // KW 1: the last block's spare waves (uniform over the wave)
    const int N = p.blob[p.o_node_off + r + 1] - p.blob[p.o_node_off + r];
    if (s >= N) return;  // uniform over the block (KW 4) or the wave (KW 1, no barriers)
    const int row = p.blob[p.o_row_off + r] + s;
    const int ns = p.n_range;
    const long rs = (long)p.total_rows * p.h_q;  // stride between ranges
    const long ri = (long)row * p.h_q + h;
    float mx = -INFINITY;
    for (int sp = KW == 4 ? t : lane; sp < ns; sp += 64 * KW) mx = fmaxf(mx, p.ws_lse[sp * rs + ri]);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if constexpr (KW == 4) {
        if (lane == 0) red[wv] = mx;
        __syncthreads();
        mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));  // finite: every node sees itself
    }
    float wsum = 0.f, a0 = 0.f, a1 = 0.f;
    auto weight = [&](float ls) { return ls == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ls - mx); };
    int sp = KW == 4 ? wv : 0;
    for (; sp + 7 * KW < ns; sp += 8 * KW) {
        float ls[8];
        float2 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            ls[u] = p.ws_lse[(sp + KW * u) * rs + ri];
            v[u] = *reinterpret_cast<const float2*>(p.ws_o + ((sp + KW * u) * rs + ri) * kAD + 2 * lane);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const float w = weight(ls[u]);
            wsum += w;
            a0 = __builtin_fmaf(w, v[u].x, a0);
            a1 = __builtin_fmaf(w, v[u].y, a1);
        }
    }
    for (; sp < ns; sp += KW) {
        const float w = weight(p.ws_lse[sp * rs + ri]);
        const float2 v = *reinterpret_cast<const float2*>(p.ws_o + (sp * rs + ri) * kAD + 2 * lane);
        wsum += w;
        a0 = __builtin_fmaf(w, v.x, a0);
        a1 = __builtin_fmaf(w, v.y, a1);
    }
    if constexpr (KW == 4) {
        part[wv][lane] = make_float2(a0, a1);
        __syncthreads();  // also orders red[] (read above) before its reuse below
        if (lane == 0) red[wv] = wsum;
        __syncthreads();
        if (wv != 0) return;
        const float2 q0 = part[0][lane], q1 = part[1][lane], q2 = part[2][lane], q3 = part[3][lane];
        wsum = ((red[0] + red[1]) + red[2]) + red[3];
        a0 = ((q0.x + q1.x) + q2.x) + q3.x;
        a1 = ((q0.y + q1.y) + q2.y) + q3.y;
    }
    const float inv = 1.f / wsum;
    reinterpret_cast<uint32_t*>(p.o + ri * kAD)[lane] = f32x2_to_bf16x2(a0 * inv, a1 * inv);
    if (lane == 0) p.lse[ri] = (mx + __log2f(wsum)) * 0.69314718055994531f;
}

// Partial results of the key ranges for lumo_tree_attention_noalloc: one fixed array
// per device, held until the process ends. Host code must not pass `scratch` itself
// to a kernel (on the host it names a stand-in, not device memory); the device
// address comes from attn_scratch() below.
static __device__ __align__(256) float scratch[LUMO_TREE_ATTENTION_SCRATCH_BYTES / sizeof(float)];

}  // namespace

hipError_t attn_scratch(float** out) {
    // one lookup per device, with that device current; the address is kept per device
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* addr[kMaxDevices] = {};
    *out = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *out = static_cast<float*>(addr[dev]);
    return hipSuccess;
}

// Row tiles per wave and key ranges of a call, the ranges at most `most`: the pair with the
// smallest estimated time, in microseconds. A block takes 64 R query rows through `each` key
// tiles, in rounds of 512 resident blocks. Measured per tile: 1.35 (R = 1) and 2.1 (R = 2) with
// at most one block per CU, 2.0 and 2.9 with two; R = 2 reads LDS half as often per product,
// so it wins where two blocks per CU compete for it (8 requests x 64 nodes x 8 heads per key
// head over 16,384 tokens, 4 ranges: 171 us, R = 1 203 us), and R = 1 on short calls, where
// fewer, longer blocks leave CUs idle (2 requests x 128 nodes, 8 heads, 1,000 tokens: 16 us, R =
// 2 20 us). A tile (32 KB of keys and values) comes from HBM once for the row chunks that
// share it, at 5.1 TB/s when the blocks fill the CUs evenly (one request of 8 key heads over
// 131,072 tokens, R = 1: 1.6 us a tile with 256 blocks, 3.3 with 512) and somewhat less otherwise. A
// round adds about 2 us around its tiles, the merge a launch and the traffic of the partial
// results, 2 x 516 B at about 5.5 TB/s per (row, head) and range: without it the 8 requests above
// took 256 ranges (2 GB of partial results) and 1,384 us. Over 58 measured shapes the choice is
// on average within 5% of the best (row tiles, ranges) pair.
AttnShape attn_shape(const lumo_attn_dims& d, const lumo_plan& pl, int max_ctx, int most) {
    constexpr long kCus = 256, kSlots = 512;
    constexpr float kTileOne[2] = {1.35f, 2.1f}, kTileTwo[2] = {2.0f, 2.9f};
    constexpr float kBlock = 2.f, kMerge = 2.f, kRange = 0.06f;
    const int rows = pl.max_nodes * (d.h_q / d.h_kv);
    const int tiles = (std::max(max_ctx, 0) + kAT - 1) / kAT + (pl.max_nodes + kAT - 1) / kAT;
    const float range = kRange + (float)pl.total_rows * (float)d.h_q * (1032.f / 5.5e6f);
    const int limit = (int)std::min<long>(std::min(most, tiles), kSlots);
    AttnShape best{1, 1};
    float best_cost = 0.f;
    for (int r = 1; r <= 2; ++r) {
        const long chunks = (rows + 16 * r * kAW - 1) / (16 * r * kAW);
        const long per = (long)d.n_req * d.h_kv * chunks;
        const float load = (kAT * kAD * 4 / 5.1e6f) / (float)chunks;  // of a block's tile, alone on HBM
        for (int n = 1; n <= limit;) {
            const int each = (tiles + n - 1) / n;
            const long blocks = n * per, rest = blocks % kSlots;
            float cost = (float)(blocks / kSlots) * ((float)each * std::max(kTileTwo[r - 1], (float)kSlots * load) + kBlock);
            if (rest) {
                const bool one = rest <= kCus;
                const float uneven = one ? 1.08f + 0.75f * (1.f - (float)rest / (float)kCus)
                                         : 1.f + 0.3f * (1.f - (float)rest / (float)kSlots);
                cost += (float)each * std::max((one ? kTileOne : kTileTwo)[r - 1], (float)rest * load * uneven) + kBlock;
            }
            if (n > 1) cost += kMerge + range * (float)n;
            if ((r == 1 && n == 1) || cost < best_cost) {
                best = {r, n};
                best_cost = cost;
            }
            if (each == 1) break;
            n = (tiles + each - 2) / (each - 1);  // the next count with fewer tiles per range
        }
    }
    return best;
}

namespace {

template <int R>
void launch_parts(AttnParams& p, int rows, hipStream_t s) {
    p.n_chunk = (rows + 16 * R * kAW - 1) / (16 * R * kAW);
    const long heads = (long)p.n_req * p.h_kv;
    // one request of 8 key/value heads over 131,072 tokens: 107.8 us with a head's ranges
    // on one XCD, 110.5 us dealt range by range; with pairs that do not fill the XCDs evenly
    // the ranges are dealt (only row chunks share keys)
    p.xcd_unit = heads % 8 == 0 ? p.n_chunk * p.n_range : p.n_chunk;
    hipLaunchKernelGGL(attn_kernel<R>, dim3((unsigned)(heads * p.n_chunk * p.n_range)), dim3(64 * kAW), 0, s, p);
}

}  // namespace

hipError_t launch_attention(const lumo_attn_dims& d, const lumo_tree_desc& desc, const AttnArgs& a, hipStream_t s) {
    const lumo_plan& pl = desc.plan;
    if (d.n_req == 0 || pl.total_nodes == 0) return hipSuccess;
    AttnParams p;
    p.blob = desc.blob;
    p.o_node_off = pl.o_node_off;
    p.o_row_off = pl.o_row_off;
    p.o_vis = pl.o_vis;
    p.ctx_off = a.ctx_off;
    p.n_req = d.n_req;
    p.h_q = d.h_q;
    p.h_kv = d.h_kv;
    p.total_rows = pl.total_rows;
    p.max_nodes = pl.max_nodes;
    p.scale_log2 = a.scale * 1.4426950408889634f;
    p.q = static_cast<const uint16_t*>(a.q);
    p.k_ctx = static_cast<const uint16_t*>(a.k_ctx);
    p.v_ctx = static_cast<const uint16_t*>(a.v_ctx);
    p.k_tree = static_cast<const uint16_t*>(a.k_tree);
    p.v_tree = static_cast<const uint16_t*>(a.v_tree);
    p.ws_o = a.ws;
    p.ws_lse = a.ws + (long)(a.n_split + 1) * pl.total_rows * d.h_q * kAD;
    p.o = static_cast<uint16_t*>(a.o);
    p.lse = a.lse;
    const int grp = d.h_q / d.h_kv;
    p.group_log2 = grp == 1 ? 0 : grp == 2 ? 1 : grp == 4 ? 2 : 3;
    const int rows = pl.max_nodes * grp;
    const AttnShape shape = attn_shape(d, pl, a.max_ctx, a.n_split + 1);  // the workspace holds n_split + 1 ranges
    p.n_range = shape.n_range;
    if (shape.row_tiles == 1)
        launch_parts<1>(p, rows, s);
    else
        launch_parts<2>(p, rows, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.n_range == 1) return e;
    const long pairs = (long)d.n_req * pl.max_nodes * d.h_q;
    // four waves per pair also where they find the device empty: one request x 16 nodes x 16
    // heads over 2,048 tokens, 11 ranges, 12.8 -> 11.0 us; 3 to 12 ranges of up to 1,024 pairs 0.94 to
    // 0.98 times as long, of 1,025 to 2,048 1.00 to 1.01 times
    if (p.n_range > 16 || (p.n_range > 3 && pairs <= 1024))
        hipLaunchKernelGGL(attn_combine_kernel<4>, dim3((unsigned)pairs), dim3(256), 0, s, p);
    else
        hipLaunchKernelGGL(attn_combine_kernel<1>, dim3((unsigned)((pairs + 3) / 4)), dim3(256), 0, s, p);
    return hipGetLastError();
}

}  // namespace lumo
