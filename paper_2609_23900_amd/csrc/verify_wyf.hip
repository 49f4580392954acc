// Tree verification in WY form for fp32 operands (d_k = d_v = 128) on the matrix cores. The
// arithmetic form is that of verify_wy.hip:
//     delta_t = beta_t (v_t - gamma_t R0 k_t) - sum_m A_m delta_{a_m},
//     o_t     = gamma_t R0 q_t + sum_m B_m delta_{a_m} + (k_t . q_t) delta_t,
// with A_m = beta_t Gamma(a_m->t) (k_{a_m} . k_t), B_m = Gamma(a_m->t) (k_{a_m} . q_t) over the
// ancestors a_m of node t.
//
// Every factor of a dot product over the keys keeps its 24 bits: x = hi + mid + lo, three
// bf16 values (hi is x rounded to bf16, mid the remainder rounded to bf16, lo what is left,
// exactly, where it is a normal number, |x| > 2^-102), and a product is the six partial products
// (hi hi, hi mid, mid hi, hi lo, lo hi, mid mid), exact in fp32. With |mid| <= 2^-8 and |lo|
// <= 2^-17 of x's power of two, what is dropped (mid lo, lo mid, lo lo) is at most 2^-24 of
// the product; with hi cut off instead of rounded it was up to 2^-22. The five small
// ones are summed first and the four steps of hi hi last, so
// that only those round at the size of the result. Six bf16 matrix instructions take 6/16 of
// the time of the fp32 ones, whose chains also round more often. Error of the
// outputs against 64-bit arithmetic: 8.6e-8 (one fp32-MFMA chain of 128 terms 1.6e-7; the
// vector-ALU kernel that served these shapes before 9.3e-8). 8 requests x 12 layers x 64 nodes x 32
// heads: 211 us (that kernel 516 us), 1 layer 28 us (148 us).
//
// A block serves (request, layer, value head) with four wavefronts of 32 state columns and
// walks the request's nodes in depth-first preorder, 32 (a chunk) at a time. The threads load
// the next chunk's key and query rows and the key rows of its path stack into registers
// during the recursion, and write the three parts to LDS when the chunk begins. Gram
// entries between the candidates (path stack, chunk) and the chunk's keys and queries, and
// R0 k and R0 q against the wave's columns, run on v_mfma_f32_16x16x32_bf16 (R0 stays in
// registers in fp32 and is split once per chunk); the coefficient records go through LDS;
// the recursion runs node by node with the deltas of the current path in registers, lane l <
// 32 forming the sum over A and the delta of its column, lane l + 32 the sum over B and the
// output. One head per block: 32-column waves hold R0 in 64 registers, which leaves room
// for the path registers at two waves per SIMD: without scratch with D = 8, with 23 to 32 spilled
// registers with D = 16 (8 x 12 layers x 64 nodes, paths of 17 nodes: 254 us; the
// vector-ALU kernel 597 us). With D = 32 the rows and records take 101 KB of LDS, one block per
// CU (one wave per SIMD; paths of 32 nodes: 434 us, the vector-ALU kernel 703 us).
#include "device_common.h"
#include "internal.h"
#include "launch.h"

namespace lumo {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kD = 128;          // d_k = d_v
constexpr int kTile = kPreChunk;  // nodes per chunk
constexpr int kCW = 32;          // state columns per wavefront
constexpr int kGS = 2 * kTile + 1;  // Gram row stride in floats: [chunk keys | chunk queries], padded
constexpr int kSlots = kD / 8;   // 16-byte slots of 8 bf16 per row and part
constexpr int kThr = 256;
static_assert(kTile == 32, "two half-chunks of 16 nodes");

struct WyfParams {
    const int32_t* blob;
    int32_t o_node_off, o_pre_row, o_pre_depth, o_pre_ci, o_chunk_off, o_chunk_stack;
    int32_t n_layers, total_rows, h_k, h_v, group;
    int32_t raw_gates;
    float qk_eps;
    const float* a_log;
    const float* dt_bias;
    const float* q;
    const float* k;
    const float* v;
    const float* g;
    const float* beta;
    const float* state0;
    float* o;
};

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 w) { return __builtin_bit_cast(bf16x8, w); }

// Two fp32 values as packed bf16 parts.
__device__ __forceinline__ void split3(float x0, float x1, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
    hi = f32x2_to_bf16x2(x0, x1);
    const float r0 = x0 - bf16_lo(hi), r1 = x1 - bf16_hi(hi);
    mid = f32x2_to_bf16x2(r0, r1);
    lo = f32x2_to_bf16x2(r0 - bf16_lo(mid), r1 - bf16_hi(mid));
}

// D path registers (8, 16 or 32), the plan's tables of 16 or 32 path-stack slots
template <int D, bool QKN>
__global__ __launch_bounds__(kThr, 2) void wyf_kernel(WyfParams p) {
    constexpr int kStack = D > kPreStack ? kDeepStack : kPreStack;
    constexpr int kCand = kStack + kTile, kTileRows = 2 * kTile + kStack, kCiWords = kStack / 4;
    constexpr int W = 16 + 2 * D;  // words per record: {-, depth, beta, f, k.q, 0, 0, 0, A[D]}, the same with B
    constexpr int kAhead = 2;  // coefficient groups requested ahead (the others on demand: registers)
    // parts of the rows [chunk keys 32 | chunk queries 32 | path-stack keys]: keys 8 c .. + 7 of
    // row n in slot c ^ (n & 15), so the 16 rows of a fragment read take 16 different slots
    __shared__ uint4 tile[3][kTileRows * kSlots];
    __shared__ __attribute__((aligned(16))) float G[kCand * kGS];
    __shared__ __attribute__((aligned(16))) float recs[kTile * W];
    __shared__ float alphas[kCand];
    __shared__ float nrm[kTileRows];  // QKN: 1/|row| of [stack keys | chunk keys | chunk queries]
    const int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the lane index is made opaque at every chunk, so that what derives from it (LDS
    // addresses) is recomputed rather than kept live across the loop
    int lane = tid & 63;
    int lq = lane & 15, lg = lane >> 4;

    // the blocks of a (request, layer) on one XCD (shared rows), the units over all of them
    int blk = xcd_units(blockIdx.x, gridDim.x, p.h_v);
    const int h = blk % p.h_v;
    blk /= p.h_v;
    const int l = blk % p.n_layers;
    const int r = blk / p.n_layers;
    const int hk = h / p.group;
    const int base = p.blob[p.o_node_off + r];
    const int N = p.blob[p.o_node_off + r + 1] - base;
    if (N <= 0) return;  // uniform over the block
    const int32_t* prow = p.blob + p.o_pre_row + base;
    const int32_t* pdep = p.blob + p.o_pre_depth + base;
    const uint32_t* pci = reinterpret_cast<const uint32_t*>(p.blob + p.o_pre_ci) + (long)kCiWords * base;
    const int32_t* stacks = p.blob + p.o_chunk_stack + (long)kStack * p.blob[p.o_chunk_off + r];
    const long krow0 = (long)l * p.total_rows;
    const bool rawg = p.raw_gates != 0;
    const float alog = rawg ? p.a_log[l * p.h_v + h] : 0.f;
    const float dtb = rawg ? p.dt_bias[l * p.h_v + h] : 0.f;
    int t = lane % kTile;  // node of this lane in the chunk views
    const int j0 = kCW * wave;
    unsigned pc = 2 * lq + (lg & 1);  // this lane's column after the exchange of the products
    bool hiB = lane >= kTile;

    // Chunk views of a lane: node t's row (positions past the end repeat the last node, so
    // that padding slots are exact copies of it), and the rows whose pieces the thread
    // stages: nodes tid / 16 and 16 + tid / 16, path-stack slots tid / 16 (+ 16); a slot past
    // the first node's depth takes the chunk's first row, never referenced.
    constexpr int kPass = kTileRows / 16;  // staged rows per thread
    struct Rows {
        int n, st[kPass - 2];  // st: node rows (2), then path-stack rows
    };
    int sr = tid >> 4, sp = tid & 15;
    auto chunk_rows = [&](int c0) {
        Rows rw;
        rw.n = prow[min(c0 + t, N - 1)];
        rw.st[0] = prow[min(c0 + sr, N - 1)];
        rw.st[1] = prow[min(c0 + 16 + sr, N - 1)];
        const int first = prow[c0];
#pragma unroll
        for (int i = 2; i < kPass - 2; ++i) {
            const int s = stacks[(c0 / kTile) * kStack + 16 * (i - 2) + sr];
            rw.st[i] = s < 0 ? first : s;
        }
        return rw;
    };
    // node t's depth, candidate slots, decay and beta; the decay of path-stack slot lane
    struct Info {
        int dep;
        uint32_t ci[D / 4];
        float gn, gs, b;
    };
    auto lane_info = [&](int c0, int row, Info& li) {
        const int pos = min(c0 + t, N - 1);
        li.dep = pdep[pos];
#pragma unroll
        for (int w = 0; w < D / 4; ++w) li.ci[w] = pci[(long)kCiWords * pos + w];
        const int s = stacks[(c0 / kTile) * kStack + (lane & (kStack - 1))];
        li.gn = p.g[(krow0 + row) * p.h_v + h];
        li.gs = p.g[(krow0 + (s < 0 ? row : s)) * p.h_v + h];
        li.b = p.beta[(krow0 + row) * p.h_v + h];
    };
    // the thread's pieces (8 elements) of its rows: keys, queries, path-stack keys
    struct Stage {
        float4 x[kPass][2];
    };
    auto stage_load = [&](const Rows& rw, Stage& sg) {
#pragma unroll
        for (int i = 0; i < kPass; ++i) {
            const float* src = (i == 2 || i == 3 ? p.q : p.k) +
                               ((krow0 + rw.st[i < 2 ? i : i - 2]) * p.h_k + hk) * kD + 8 * sp;
            sg.x[i][0] = *reinterpret_cast<const float4*>(src);
            sg.x[i][1] = *reinterpret_cast<const float4*>(src + 4);
        }
    };
    auto stage_store = [&](const Stage& sg) {
#pragma unroll
        for (int i = 0; i < kPass; ++i) {
            const int row = 16 * i + sr;
            const float4 a = sg.x[i][0], b = sg.x[i][1];
            uint32_t hi[4], mid[4], lo[4];
            split3(a.x, a.y, hi[0], mid[0], lo[0]);
            split3(a.z, a.w, hi[1], mid[1], lo[1]);
            split3(b.x, b.y, hi[2], mid[2], lo[2]);
            split3(b.z, b.w, hi[3], mid[3], lo[3]);
            const int at = row * kSlots + (sp ^ (row & 15));
            tile[0][at] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            tile[1][at] = make_uint4(mid[0], mid[1], mid[2], mid[3]);
            tile[2][at] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            if constexpr (QKN) {  // the row's 16 threads are 16 adjacent lanes
                float ss = 0.f;
                const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) ss = __builtin_fmaf(v[e], v[e], ss);
                ss += __shfl_xor(ss, 1);
                ss += __shfl_xor(ss, 2);
                ss += __shfl_xor(ss, 4);
                ss += __shfl_xor(ss, 8);
                if (sp == 0)
                    nrm[row < kTile ? kStack + row : row < 2 * kTile ? kCand + (row - kTile) : row - 2 * kTile] =
                        __builtin_amdgcn_rsqf(ss + p.qk_eps);
            }
        }
    };
    auto lds_barrier = [&]() {  // no wait for global memory operations
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // part x of keys 32 kb + 8 lg .. + 7 of tile row `row`
    auto frag = [&](int x, int row, int kb) -> bf16x8 {
        return as_bf16x8(tile[x][row * kSlots + ((4 * kb + lg) ^ (row & 15))]);
    };
    auto mfma = [](bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); };

    Rows rowC = chunk_rows(0), rowA = rowC;
    if (N > kTile) rowA = chunk_rows(kTile);
    Stage stg;
    stage_load(rowC, stg);
    Info info;
    lane_info(0, rowC.n, info);
    // R0 as B fragments of the 16x16x32 products: column n = lane % 16 of tile ct is state
    // column j0 + 2 n + ct, key block kb holds keys 32 kb + 8 (lane / 16) + e
    float R0[2][kD / 32][8];
    {
        const float* S = p.state0 + (((long)r * p.n_layers + l) * p.h_v + h) * (long)(kD * kD) + (long)(8 * lg) * kD + j0 +
                         2 * lq;
#pragma unroll
        for (int kb = 0; kb < kD / 32; ++kb)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float2 w = *reinterpret_cast<const float2*>(S + (long)(32 * kb + e) * kD);
                R0[0][kb][e] = w.x;
                R0[1][kb][e] = w.y;
            }
    }
    // delta of the current path by depth; a node at depth D (17 nodes per path, D = 16) has
    // no descendants
    constexpr int kDst = D < 32 ? D + 1 : D;
    float dst[kDst];
#pragma unroll
    for (int m = 0; m < kDst; ++m) dst[m] = 0.f;

    // Columns whose delta was not finite at some node: a slot at a node's depth or below may
    // then hold another branch's NaN or infinity, which must not reach the node through a
    // zero coefficient.
    uint64_t spoilt = 0;

    // largest magnitude of z and x's entries, NaN if one is
    auto largest = [](float z, const f32x4& x) {
#pragma unroll
        for (int i = 0; i < 4; ++i) z = __builtin_elementwise_maximum(z, __builtin_fabsf(x[i]));
        return z;
    };
    // this lane's keys 32 kb + 8 lg + e of a row; finite entries of x, the others from y
    auto whole_row = [&](const float* mat, int row) { return mat + ((krow0 + row) * p.h_k + hk) * kD + 8 * lg; };
    auto keep_finite = [](f32x4& x, const f32x4& y) {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = __builtin_fabsf(x[i]) < INFINITY ? x[i] : y[i];
    };
    // R0 [k | q] of the chunk's two halves of 16 nodes: x[hf][0], [1] the k products of column
    // tiles 0, 1, x[hf][2], [3] the q products; after the 4 x 4 exchange of lane groups
    // (permlane32, then permlane16 swaps) lane l < 32 holds in x[hf][b][i] R0 k, lane l + 32
    // R0 q, of node 16 hf + 4 b + i and column j0 + pc.
    auto products = [&](bool two, f32x4 (&x)[2][4]) {
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
            for (int c = 0; c < 4; ++c) x[hf][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < kD / 32; ++kb) {  // the five small partial products
            bf16x8 rh[2], rm[2], rl[2];
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) {
                uint32_t hi[4], mid[4], lo[4];
                // opaque per chunk: otherwise the parts of all key blocks are computed once
                // before the chunk loop and kept (96 registers that are not there)
#pragma unroll
                for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(R0[ct][kb][e]));
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    split3(R0[ct][kb][2 * e], R0[ct][kb][2 * e + 1], hi[e], mid[e], lo[e]);
                rh[ct] = as_bf16x8(make_uint4(hi[0], hi[1], hi[2], hi[3]));
                rm[ct] = as_bf16x8(make_uint4(mid[0], mid[1], mid[2], mid[3]));
                rl[ct] = as_bf16x8(make_uint4(lo[0], lo[1], lo[2], lo[3]));
            }
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                if (hf == 1 && !two) break;  // uniform
#pragma unroll
                for (int kq = 0; kq < 2; ++kq) {
                    const int row = kTile * kq + 16 * hf + lq;
                    const bf16x8 fh = frag(0, row, kb), fm = frag(1, row, kb), fl = frag(2, row, kb);
#pragma unroll
                    for (int ct = 0; ct < 2; ++ct) {
                        f32x4& a = x[hf][2 * kq + ct];
                        a = mfma(fl, rh[ct], a);
                        a = mfma(fm, rm[ct], a);
                        a = mfma(fh, rl[ct], a);
                        a = mfma(fm, rh[ct], a);
                        a = mfma(fh, rm[ct], a);
                    }
                }
            }
            asm volatile("" ::: "memory");  // one key block's fragments at a time (registers)
        }
#pragma unroll
        for (int kb = 0; kb < kD / 32; ++kb) {  // hi hi
            bf16x8 rh[2];
#pragma unroll
            for (int ct = 0; ct < 2; ++ct) {
                uint32_t hi[4];
#pragma unroll
                for (int e = 0; e < 8; ++e) asm volatile("" : "+v"(R0[ct][kb][e]));
#pragma unroll
                for (int e = 0; e < 4; ++e) hi[e] = f32x2_to_bf16x2(R0[ct][kb][2 * e], R0[ct][kb][2 * e + 1]);
                rh[ct] = as_bf16x8(make_uint4(hi[0], hi[1], hi[2], hi[3]));
            }
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                if (hf == 1 && !two) break;
#pragma unroll
                for (int kq = 0; kq < 2; ++kq) {
                    const bf16x8 fh = frag(0, kTile * kq + 16 * hf + lq, kb);
#pragma unroll
                    for (int ct = 0; ct < 2; ++ct) x[hf][2 * kq + ct] = mfma(fh, rh[ct], x[hf][2 * kq + ct]);
                }
            }
            asm volatile("" ::: "memory");
        }
    };
    // An infinite factor has no three parts (its remainder is NaN, and it meets zero and
    // opposite parts of the other factor), and one next to the largest float rounds up to one:
    // products of half hf that are not finite are taken again from the whole values, on the
    // fp32 matrix instructions.
    auto recheck = [&](int hf, int rowN, f32x4 (&x)[4]) {
        float z = 0.f;
#pragma unroll
        for (int c = 0; c < 4; ++c) z = largest(z, x[c]);
        if (__ballot(!(z < INFINITY)) == 0) return;  // uniform
        const int row = __shfl(rowN, 16 * hf + lq);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float* src = whole_row(c < 2 ? p.k : p.q, row);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < kD / 32; ++kb)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(src[32 * kb + e], R0[c & 1][kb][e], acc, 0, 0, 0);
            keep_finite(x[c], acc);
        }
    };
    auto exchange = [&](f32x4 (&x)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[c][i]), __float_as_uint(x[c + 2][i]),
                                                                 false, false);
                x[c][i] = __uint_as_float(sw[0]);
                x[c + 2][i] = __uint_as_float(sw[1]);
            }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 4; c += 2) {
                const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(x[c][i]), __float_as_uint(x[c + 1][i]),
                                                                 false, false);
                x[c][i] = __uint_as_float(sw[0]);
                x[c + 1][i] = __uint_as_float(sw[1]);
            }
    };

    for (int c0 = 0; c0 < N; c0 += kTile) {
        const bool more = c0 + kTile < N;
        const bool two = c0 + kTile / 2 < N;  // the second half holds real nodes
        const int rowN = rowC.n;  // this chunk's row of node t
        asm volatile("" : "+v"(lane));
        lq = lane & 15;
        lg = lane >> 4;
        t = lane % kTile;
        hiB = lane >= kTile;
        pc = 2 * lq + (lg & 1);
        sr = 4 * wave + lg;
        sp = lq;
        stage_store(stg);  // (every wave has read the previous chunk's rows: barrier below)
        if (wave == 0) {  // decays of the candidates
            const float an = __expf(rawg ? raw_log_alpha(info.gn, alog, dtb) : info.gn);
            const float as = __expf(rawg ? raw_log_alpha(info.gs, alog, dtb) : info.gs);
            if (lane < kTile) alphas[kStack + lane] = an;
            if (lane < kStack) alphas[lane] = as;
        }
        lds_barrier();  // the chunk's rows and decays are complete
        // the wave's values of a half (lower lanes: column j0 + pc)
        float val[16];
        auto load_values = [&](int hf) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int rn = __builtin_amdgcn_readlane(rowN, 16 * hf + i);
                const float* row = p.v + ((krow0 + rn) * p.h_v + h) * kD + j0;  // uniform
                val[i] = row[pc];
            }
        };
        // ---- Gram: wave w takes columns 16 w .. + 15 of [chunk keys | chunk queries]
        {
            constexpr int kRT = kCand / 16;  // row tiles: path stack, then the chunk's keys
            f32x4 small[kRT], big[kRT];
#pragma unroll
            for (int i = 0; i < kRT; ++i) small[i] = big[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < kD / 32; ++kb) {
                const int col = 16 * wave + lq;
                const bf16x8 bh = frag(0, col, kb), bm = frag(1, col, kb), bl = frag(2, col, kb);
#pragma unroll
                for (int i = 0; i < kRT; ++i) {
                    const int row = (16 * i < kStack ? 2 * kTile + 16 * i : 16 * i - kStack) + lq;
                    const bf16x8 ah = frag(0, row, kb), am = frag(1, row, kb), al = frag(2, row, kb);
                    small[i] = mfma(al, bh, small[i]);
                    small[i] = mfma(am, bm, small[i]);
                    small[i] = mfma(ah, bl, small[i]);
                    small[i] = mfma(am, bh, small[i]);
                    small[i] = mfma(ah, bm, small[i]);
                    big[i] = mfma(ah, bh, big[i]);
                }
                asm volatile("" ::: "memory");
            }
            float z = 0.f;
#pragma unroll
            for (int i = 0; i < kRT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) small[i][e] += big[i][e];
#pragma unroll
            for (int i = 0; i < kRT; ++i) z = largest(z, small[i]);
            if (__ballot(!(z < INFINITY))) {  // uniform: as for R0 [k | q] (recheck)
                const float* cs = whole_row(wave < 2 ? p.k : p.q, __shfl(rowN, (16 * wave + lq) % kTile));
#pragma unroll
                for (int i = 0; i < kRT; ++i) {
                    int row = __shfl(rowN, (16 * i + kStack + lq) % kTile);  // a node of the chunk
                    if (16 * i < kStack) {
                        const int s = stacks[(c0 / kTile) * kStack + 16 * i + lq];
                        row = s < 0 ? prow[c0] : s;
                    }
                    const float* rs = whole_row(p.k, row);
                    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kb = 0; kb < kD / 32; ++kb)
#pragma unroll
                        for (int e = 0; e < 8; ++e)
                            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(rs[32 * kb + e], cs[32 * kb + e], acc, 0, 0, 0);
                    keep_finite(small[i], acc);
                }
            }
#pragma unroll
            for (int i = 0; i < kRT; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) G[(16 * i + 4 * lg + e) * kGS + 16 * wave + lq] = small[i][e];
        }
        f32x4 px[2][4];
        products(two, px);
        lds_barrier();  // the Gram is complete, and every wave has read the rows

        // ---- coefficient records (lanes 0..31: A, lanes 32..63: B), a quarter of the chunk's
        // nodes per wave would idle lanes: the first wave writes them all
        if (wave == 0) {
            const float* Gc = G + (hiB ? kTile : 0) + t;
            const float bt = rawg ? raw_beta(info.b) : info.b;
            float nk = 1.f, nq = 1.f;
            if constexpr (QKN) {
                nk = nrm[kStack + t];
                nq = nrm[kCand + t];
            }
            const float sc = hiB ? nq : bt * nk;
            float gam = alphas[kStack + t];  // Gamma(a_{d-1} -> t) = alpha_t
            float cv[D];
#pragma unroll
            for (int m = D - 1; m >= 0; --m) {
                // past the depth candidate 0 is read and masked, so the reads go out together
                const bool live = m < info.dep;
                const int ci = live ? (int)((info.ci[m / 4] >> (8 * (m % 4))) & 0xffu) : 0;
                float gv = Gc[ci * kGS];
                if constexpr (QKN) gv *= nrm[ci];
                const float av = alphas[ci];
                cv[m] = live ? (sc * gam) * gv : 0.f;
                gam *= live ? av : 1.f;  // then Gamma(a_{m-1} -> t); finally gamma_t
            }
            float* rt = recs + t * W + (hiB ? 8 + D : 0);
#pragma unroll
            for (int q4 = 0; q4 < D / 4; ++q4)
                *reinterpret_cast<float4*>(rt + 8 + 4 * q4) =
                    make_float4(cv[4 * q4], cv[4 * q4 + 1], cv[4 * q4 + 2], cv[4 * q4 + 3]);
            *reinterpret_cast<float4*>(rt) = make_float4(0.f, __int_as_float(info.dep), bt,
                                                         hiB ? gam * nq : -(gam * nk));
            *reinterpret_cast<float4*>(rt + 4) = make_float4(G[(kStack + t) * kGS + kTile + t] * (nk * nq), 0.f, 0.f, 0.f);
        }
        if (more) {  // the next chunk's lane view lands during the recursion
            rowC = rowA;
            lane_info(c0 + kTile, rowC.n, info);
        }
        lds_barrier();  // the records are written

        struct Head {
            float4 w0, c[kAhead];
            float kq;
        };
        auto load_head = [&](int n, Head& hd) {
            const float* cf = recs + n * W + (hiB ? 8 + D : 0);
            hd.w0 = *reinterpret_cast<const float4*>(cf);
            hd.kq = cf[4];
#pragma unroll
            for (int g = 0; g < kAhead; ++g) hd.c[g] = *reinterpret_cast<const float4*>(cf + 8 + 4 * g);
        };
        // Straight-line over the 16 nodes of a half (padding slots recompute the last node
        // exactly). A node's record is taken into registers before the next one is requested.
        // The upper half's outputs replace the values in `val` and are stored at the end.
        auto recursion = [&](int hf, const f32x4 (&px)[4]) {
            Head nx;
            load_head(16 * hf, nx);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int n = 16 * hf + i;
#pragma unroll
                for (int g = 0; g < kAhead; ++g)
                    asm volatile("" ::"v"(nx.c[g].x), "v"(nx.c[g].y), "v"(nx.c[g].z), "v"(nx.c[g].w));
                asm volatile("" ::"v"(nx.w0.y), "v"(nx.w0.z), "v"(nx.w0.w), "v"(nx.kq) : "memory");
                const Head cu = nx;
                if (i + 1 < 16) load_head(n + 1, nx);
                const int d = __builtin_amdgcn_readfirstlane(__float_as_int(cu.w0.y));  // uniform
                float s0 = 0.f, s1 = 0.f;
                const float* cl = recs + n * W + (hiB ? 8 + D : 0) + 8;
                if (spoilt) {  // uniform: depth by depth, nothing past the node's own
                    for (int m = 0; m < d; ++m) {
                        const float x = cl[m];
                        if (m & 1)
                            s1 = __builtin_fmaf(x, dst[m], s1);
                        else
                            s0 = __builtin_fmaf(x, dst[m], s0);
                    }
                } else {  // four depths at a time: the entries past the depth are zero
#pragma unroll
                    for (int g = 0; g < kAhead; ++g) {
                        if (g > 0 && d <= 4 * g) break;  // uniform
                        s0 = __builtin_fmaf(cu.c[g].x, dst[4 * g], s0);
                        s1 = __builtin_fmaf(cu.c[g].y, dst[4 * g + 1], s1);
                        s0 = __builtin_fmaf(cu.c[g].z, dst[4 * g + 2], s0);
                        s1 = __builtin_fmaf(cu.c[g].w, dst[4 * g + 3], s1);
                    }
                    if constexpr (kAhead < D / 4) {
#pragma unroll
                        for (int g0 = kAhead; g0 < D / 4; g0 += 2) {
                            if (d <= 4 * g0) break;
                            float4 c2[2];
#pragma unroll
                            for (int x = 0; x < 2; ++x) c2[x] = *reinterpret_cast<const float4*>(cl + 4 * (g0 + x));
#pragma unroll
                            for (int x = 0; x < 2; ++x) {
                                const int g = g0 + x;
                                s0 = __builtin_fmaf(c2[x].x, dst[4 * g], s0);
                                s1 = __builtin_fmaf(c2[x].y, dst[4 * g + 1], s1);
                                s0 = __builtin_fmaf(c2[x].z, dst[4 * g + 2], s0);
                                s1 = __builtin_fmaf(c2[x].w, dst[4 * g + 3], s1);
                            }
                        }
                    }
                }
                const float sm = s0 + s1;
                // lower half: v - gamma R0 k, then delta = beta u - sum A; upper half:
                // gamma_q R0 q + sum B, then the output with the lower half's delta
                const float u = __builtin_fmaf(cu.w0.w, px[i / 4][i % 4], hiB ? sm : val[i]);
                const float da = __builtin_fmaf(cu.w0.z, u, -sm);
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(da), __float_as_uint(da), false, false);
                const float delta = __uint_as_float(sw[0]);
                dst[d < kDst ? d : kDst - 1] = delta;
                spoilt |= __ballot(!(__builtin_fabsf(delta) < INFINITY));
                val[i] = __builtin_fmaf(cu.kq, delta, u);
            }
            if (hiB) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int rn = __builtin_amdgcn_readlane(rowN, 16 * hf + i);
                    float* row = p.o + ((krow0 + rn) * p.h_v + h) * kD + j0;  // uniform
                    row[pc] = val[i];
                }
            }
        };
        load_values(0);
        recheck(0, rowN, px[0]);
        exchange(px[0]);
        recursion(0, px[0]);
        if (two) {
            load_values(1);
            // the next chunk's rows, behind the values (only now are there registers for them)
            if (more) stage_load(rowC, stg);
            recheck(1, rowN, px[1]);
            exchange(px[1]);
            recursion(1, px[1]);
        }
        if (c0 + 2 * kTile < N) rowA = chunk_rows(c0 + 2 * kTile);
    }
}

template <int D>
void launch_d(const WyfParams& p, long nb, bool qkn, hipStream_t s) {
    if (qkn)
        hipLaunchKernelGGL((wyf_kernel<D, true>), dim3((unsigned)nb), dim3(kThr), 0, s, p);
    else
        hipLaunchKernelGGL((wyf_kernel<D, false>), dim3((unsigned)nb), dim3(kThr), 0, s, p);
}

}  // namespace

hipError_t launch_wyf(const lumo_gdn_dims& d, const lumo_tree_desc& desc, const GdnArgs& a, hipStream_t s) {
    const lumo_plan& pl = desc.plan;
    if (pl.total_nodes == 0) return hipSuccess;
    WyfParams p;
    p.blob = desc.blob;
    p.o_node_off = pl.o_node_off;
    p.o_pre_row = pl.o_pre_row;
    p.o_pre_depth = pl.o_pre_depth;
    p.o_pre_ci = pl.o_pre_ci;
    p.o_chunk_off = pl.o_chunk_off;
    p.o_chunk_stack = pl.o_chunk_stack;
    p.n_layers = d.n_layers;
    p.total_rows = pl.total_rows;
    p.h_k = d.h_k;
    p.h_v = d.h_v;
    p.group = d.h_v / d.h_k;
    p.raw_gates = (a.prep.flags & LUMO_PREP_RAW_GATES) != 0;
    p.qk_eps = a.prep.qk_eps;
    p.a_log = a.prep.a_log;
    p.dt_bias = a.prep.dt_bias;
    p.q = static_cast<const float*>(a.q);
    p.k = static_cast<const float*>(a.k);
    p.v = static_cast<const float*>(a.v);
    p.g = a.g;
    p.beta = a.beta;
    p.state0 = a.state0;
    p.o = static_cast<float*>(a.o);
    const bool qkn = (a.prep.flags & LUMO_PREP_QK_NORM) != 0;
    const long nb = (long)d.n_req * d.n_layers * d.h_v;
    if (pl.max_depth <= 9) {
        launch_d<8>(p, nb, qkn, s);
    } else if (pl.max_depth <= kWyMaxDepth) {
        launch_d<16>(p, nb, qkn, s);
    } else {
        const int64_t section = deep_section(pl, desc.host_blob);
        if (section < 0) return hipErrorNotSupported;
        p.o_pre_ci = (int32_t)section + kDeepHead;
        p.o_chunk_stack = p.o_pre_ci + kDeepStack / 4 * pl.total_nodes;
        launch_d<32>(p, nb, qkn, s);
    }
    return hipGetLastError();
}

}  // namespace lumo
