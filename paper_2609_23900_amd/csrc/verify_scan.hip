// Path-parallel tree verification by sequential path scans (LumoTree Sec. IV-A,
// Alg. 2; Eq. (2)-(3)), in two forms that give the same bits: level by level through cut
// states in the workspace (scan_kernel), and the whole tree in one launch with the
// states it returns to in registers (scan_tree_kernel, below).
//
// scan_kernel: one wavefront per (segment, layer, value head, 64-wide value tile). Each lane owns
// one value row j of the head matrix R (the full key dimension, d_k fp32 values, in
// VGPRs) and carries it through every node of its segment: the state tile is loaded
// once (pre-tree state or an exported cut state) and reused across the path loop.
// Rows of R evolve independently, so the k.R and R.q contractions are lane-local;
// the node's k and q rows are wave-uniform and are read with scalar loads.
// Segments of a dependency level are independent and run in one launch; a segment
// exports its tile to the workspace at nodes whose other children start segments of
// the next level (cut states, Sec. IV-C, Eq. (4)). With operand preparation (Sec.
// IV-B) the gates come from raw inputs and the key and query rows are used divided by
// sqrt(|x|^2 + eps), computed as the commit's replay computes them.
#include "device_common.h"
#include "dispatch.h"
#include "internal.h"
#include "launch.h"

namespace lumo {
namespace {

// Pointers are separate __restrict__ kernel arguments so that the compiler may read
// the wave-uniform key and query rows with scalar loads.
struct ScanParams {
    const int32_t* blob;
    int32_t o_seg, o_seg_nodes;
    int32_t n_layers, total_rows, h_k, h_v, d_v, group, n_vtiles;
    int32_t seg_first;
    PrepArgs prep;  // operand preparation (Sec. IV-B); flags 0 = operands as given
};

template <int DK, int OPT>
__global__ __launch_bounds__(64) void scan_kernel(ScanParams p, const typename Op<OPT>::T* __restrict__ q,
                                                  const typename Op<OPT>::T* __restrict__ k,
                                                  const typename Op<OPT>::T* __restrict__ v,
                                                  const float* __restrict__ g, const float* __restrict__ gbeta,
                                                  const float* __restrict__ state0,
                                                  typename Op<OPT>::T* __restrict__ o,
                                                  float* __restrict__ node_states, float* __restrict__ ws) {
    int t = xcd_remap(blockIdx.x, gridDim.x);
    const int vt = t % p.n_vtiles;
    t /= p.n_vtiles;
    const int h = t % p.h_v;
    t /= p.h_v;
    const int l = t % p.n_layers;
    const int s = p.seg_first + t / p.n_layers;

    const int j = vt * 64 + (int)threadIdx.x;
    const bool act = j < p.d_v;
    const int jc = act ? j : p.d_v - 1;
    const int hk = h / p.group;
    const int32_t* seg = p.blob + p.o_seg + kSegWords * s;
    const int req = seg[0], src = seg[1], first = seg[2], len = seg[3];
    const long mat = (long)DK * p.d_v;

    const float* S0 = src < 0 ? state0 + (((long)req * p.n_layers + l) * p.h_v + h) * mat
                              : ws + (((long)src * p.n_layers + l) * p.h_v + h) * mat;
    float S[DK];
#pragma unroll
    for (int i = 0; i < DK; ++i) S[i] = S0[(long)i * p.d_v + jc];

    const bool qkn = (p.prep.flags & LUMO_PREP_QK_NORM) != 0;  // uniform
    const bool rawg = (p.prep.flags & LUMO_PREP_RAW_GATES) != 0;
    const float alog = rawg ? p.prep.a_log[l * p.h_v + h] : 0.f;
    const float dtb = rawg ? p.prep.dt_bias[l * p.h_v + h] : 0.f;
    for (int e = first; e < first + len; ++e) {
        const int32_t* en = p.blob + p.o_seg_nodes + kSegNodeWords * e;
        const int row = en[0], wout = en[1], cut = en[2];
        const long gi = ((long)l * p.total_rows + row) * p.h_v + h;
        const long ki = (((long)l * p.total_rows + row) * p.h_k + hk) * DK;
        const float gv = g[gi], bv = gbeta[gi];
        const float alpha = __expf(rawg ? raw_log_alpha(gv, alog, dtb) : gv);
        const float beta = rawg ? raw_beta(bv) : bv;
        const float vj = Op<OPT>::ld(v, gi * p.d_v + jc);
        const float ks = qkn ? row_rsq_norm<DK, OPT>(k + ki, p.prep.qk_eps) : 1.f;
        gdn_row_update<DK, OPT>(S, k + ki, vj, alpha, beta, ks);
        if (wout) {
            const float qs = qkn ? row_rsq_norm<DK, OPT>(q + ki, p.prep.qk_eps) : 1.f;
            const float ov = gdn_row_output<DK, OPT>(S, q + ki, qs);
            if (act) {
                Op<OPT>::st(o, gi * p.d_v + j, ov);
                if (node_states) {
                    float* dst = node_states + gi * mat;
#pragma unroll
                    for (int i = 0; i < DK; ++i) dst[(long)i * p.d_v + j] = S[i];
                }
            }
        }
        if (cut >= 0 && act) {
            float* dst = ws + (((long)cut * p.n_layers + l) * p.h_v + h) * mat;
#pragma unroll
            for (int i = 0; i < DK; ++i) dst[(long)i * p.d_v + j] = S[i];
        }
    }
}

// The same scan in one launch, without cut states in memory. The level-by-level schedules
// above move every cut state to the workspace and back (a 64-node tree: 19 stores and 37
// loads of a 64 KB tile per value head; the batched workload 48 GB per call against 1.4 GB
// of operands and states, at 5 TB/s). Here a wavefront takes 16 value columns through the
// whole tree, depth first, and keeps the states it returns to in registers: with the
// child that needs most of them visited last a tree needs at most log2(leaves) saved
// states (plan.cpp), and a column tile this narrow leaves room for NS of them (d_k = 128, NS = 4:
// 242 registers and no scratch with packed fp32 instructions off; with them on 77 to 107 spill).
//
// Lane 4 c + r holds the keys i = r (mod 4) of column c: element i of a dot product goes
// into partial sum i % 4 (Dot4), so each lane owns one of the four chains of its column
// and two quad exchanges add them in Dot4's order. Every value is computed with the
// operations, and in the order, of scan_kernel, so the outputs are the same bits.
//
// A block is four such wavefronts of one key head ((value head, 16-column tile) pairs),
// which share the key and query rows: chunks of kScanChunk visited nodes, converted to
// fp32 and split by i % 4 on the way into LDS, one chunk ahead of their use. Bound by the
// vector ALUs (128 of about 190 instructions per node and wave are the recurrence's fma
// and mul at d_k = 128) with the LDS port next (the rows are read by every wave).
constexpr int kScanChunk = 16;

struct ScanTreeParams {
    const int32_t* blob;
    int32_t o_node_off, o_order;
    int32_t n_layers, total_rows, h_k, h_v, d_v, group, n_ct, nwk, n_wb;
};

template <int DK, int OPT, int NS>
__global__ __launch_bounds__(256, 2) void scan_tree_kernel(ScanTreeParams p,
                                                           const typename Op<OPT>::T* __restrict__ q,
                                                           const typename Op<OPT>::T* __restrict__ k,
                                                           const typename Op<OPT>::T* __restrict__ v,
                                                           const float* __restrict__ g, const float* __restrict__ gbeta,
                                                           const float* __restrict__ state0,
                                                           typename Op<OPT>::T* __restrict__ o) {
    using T = typename Op<OPT>::T;
    constexpr int KC = kScanChunk;
    constexpr int E = DK / 4;    // keys per lane
    constexpr int RS = E + 4;    // floats per residue row (padded: the four rows on different banks)
    constexpr int EPT = DK / 16;  // row elements a thread stages (16 threads per node)
    struct __attribute__((aligned(EPT * sizeof(T)))) Piece {
        T e[EPT];
    };
    __shared__ __attribute__((aligned(16))) float rows[2][KC][2][4 * RS];  // [buffer][node][key, query]
    __shared__ __attribute__((aligned(16))) float4 heads[2][4][KC];        // per wave: {alpha, beta, row, code}
    __shared__ __attribute__((aligned(16))) float vals[2][4][KC][16];      // per wave: values, then outputs
    const int tid = (int)threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;

    // the blocks of a (request, layer) on one XCD (shared rows), the units over all of them
    int blk = xcd_units(blockIdx.x, gridDim.x, p.h_k * p.n_wb);
    const int wb = blk % p.n_wb;
    blk /= p.n_wb;
    const int hk = blk % p.h_k;
    blk /= p.h_k;
    const int l = blk % p.n_layers;
    const int r = blk / p.n_layers;
    const int base = p.blob[p.o_node_off + r];
    const int N = p.blob[p.o_node_off + r + 1] - base;
    if (N <= 0) return;  // uniform over the block
    const int gw = wb * 4 + wave;
    const bool wact = gw < p.nwk;  // uniform: idle waves stage rows only
    const int h = hk * p.group + (wact ? gw / p.n_ct : 0);
    const int j0 = (wact ? gw % p.n_ct : 0) * 16;
    const int c = lane >> 2, res = lane & 3;
    const int2* order = reinterpret_cast<const int2*>(p.blob + p.o_order) + base;
    const long lrow = (long)l * p.total_rows;

    float S[E];
    {
        const float* S0 = state0 + (((long)r * p.n_layers + l) * p.h_v + h) * (long)DK * p.d_v + (long)res * p.d_v + j0 + c;
#pragma unroll
        for (int t = 0; t < E; ++t) S[t] = S0[(long)(4 * t) * p.d_v];
    }
    float saved[NS][E];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int t = 0; t < E; ++t) saved[s][t] = 0.f;

    // Staging of the chunk at c0: thread tid carries elements EPT (tid % 16) .. of node
    // tid / 16's key and query rows; lane (n = lane / 4, columns 4 (lane % 4) ..) its
    // wave's values of node n and, once per node, gates and code. Positions past the end
    // repeat the last node (staged, never visited).
    struct Regs {
        Piece kp, qp;
        T vv[4];
        float gv, bv;
        int2 en;
    };
    const int sn = tid >> 4, sp = tid & 15;
    auto fetch = [&](int2 block_en, int2 wave_en, Regs& x) {
        const long kr = ((lrow + block_en.x) * p.h_k + hk) * DK + EPT * sp;
        x.kp = *reinterpret_cast<const Piece*>(k + kr);
        x.qp = *reinterpret_cast<const Piece*>(q + kr);
        const long gi = (lrow + wave_en.x) * p.h_v + h;
        x.gv = g[gi];
        x.bv = gbeta[gi];
        struct __attribute__((aligned(4 * sizeof(T)))) V4 {
            T e[4];
        };
        const V4 w = *reinterpret_cast<const V4*>(v + gi * p.d_v + j0 + 4 * res);
#pragma unroll
        for (int e = 0; e < 4; ++e) x.vv[e] = w.e[e];
        x.en = wave_en;
    };
    auto store = [&](const Regs& x, int buf) {
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int i = EPT * sp + e;
            rows[buf][sn][0][(i & 3) * RS + (i >> 2)] = Op<OPT>::ld(x.kp.e, e);
            rows[buf][sn][1][(i & 3) * RS + (i >> 2)] = Op<OPT>::ld(x.qp.e, e);
        }
        *reinterpret_cast<float4*>(&vals[buf][wave][c][4 * res]) =
            make_float4(Op<OPT>::ld(x.vv, 0), Op<OPT>::ld(x.vv, 1), Op<OPT>::ld(x.vv, 2), Op<OPT>::ld(x.vv, 3));
        if (res == 0)
            heads[buf][wave][c] = make_float4(__expf(x.gv), x.bv, __int_as_float(x.en.x), __int_as_float(x.en.y));
    };
    auto entry = [&](int pos) { return order[min(pos, N - 1)]; };

    Regs nx;
    fetch(entry(sn), entry(c), nx);
    store(nx, 0);
    int2 ebn = entry(KC + sn), ewn = entry(KC + c);
    __syncthreads();
    for (int c0 = 0, buf = 0; c0 < N; c0 += KC, buf ^= 1) {
        const bool more = c0 + KC < N;
        if (more) {
            fetch(ebn, ewn, nx);
            ebn = entry(c0 + 2 * KC + sn);
            ewn = entry(c0 + 2 * KC + c);
        }
        const int cnt = min(N - c0, KC);
        if (wact) {
            for (int n = 0; n < cnt; ++n) {
                const float4 hd = heads[buf][wave][n];
                const int code = __builtin_amdgcn_readfirstlane(__float_as_int(hd.w));
                const float alpha = hd.x, beta = hd.y;
                const float vj = vals[buf][wave][n][c];
                const float* kr = &rows[buf][n][0][res * RS];
                const float* qr = &rows[buf][n][1][res * RS];
                const int src = code & 0xff, save = code >> 8;  // uniform
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    if (src == 2 + s) {
#pragma unroll
                        for (int t = 0; t < E; ++t) S[t] = saved[s][t];
                    }
                float kf[E];
#pragma unroll
                for (int t = 0; t < E; t += 4) {
                    const float4 w = *reinterpret_cast<const float4*>(kr + t);
                    kf[t] = w.x;
                    kf[t + 1] = w.y;
                    kf[t + 2] = w.z;
                    kf[t + 3] = w.w;
                }
                float u = 0.f;
#pragma unroll
                for (int t = 0; t < E; ++t) u = __builtin_fmaf(S[t], kf[t], u);
                u = quad_sum(u);
                const float delta = beta * __builtin_fmaf(-alpha, u, vj);
                float ov = 0.f;
#pragma unroll
                for (int t = 0; t < E; t += 4) {
                    const float4 w = *reinterpret_cast<const float4*>(qr + t);
                    S[t] = __builtin_fmaf(delta, kf[t], alpha * S[t]);
                    S[t + 1] = __builtin_fmaf(delta, kf[t + 1], alpha * S[t + 1]);
                    S[t + 2] = __builtin_fmaf(delta, kf[t + 2], alpha * S[t + 2]);
                    S[t + 3] = __builtin_fmaf(delta, kf[t + 3], alpha * S[t + 3]);
                    ov = __builtin_fmaf(S[t], w.x, ov);
                    ov = __builtin_fmaf(S[t + 1], w.y, ov);
                    ov = __builtin_fmaf(S[t + 2], w.z, ov);
                    ov = __builtin_fmaf(S[t + 3], w.w, ov);
                }
                ov = quad_sum(ov);
                vals[buf][wave][n][c] = ov;  // the quad's four lanes write the same value
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    if (save == 1 + s) {
#pragma unroll
                        for (int t = 0; t < E; ++t) saved[s][t] = S[t];
                    }
            }
            // the chunk's outputs of this wave: node lane / 4, columns 4 (lane % 4) ..
            if (c < cnt) {
                const float4 w = *reinterpret_cast<const float4*>(&vals[buf][wave][c][4 * res]);
                const int row = __float_as_int(heads[buf][wave][c].z);
                T* dst = o + ((lrow + row) * p.h_v + h) * p.d_v + j0 + 4 * res;
                if constexpr (OPT == 1)
                    *reinterpret_cast<uint2*>(dst) = make_uint2(f32x2_to_bf16x2(w.x, w.y), f32x2_to_bf16x2(w.z, w.w));
                else
                    *reinterpret_cast<float4*>(dst) = w;
            }
        }
        if (more) store(nx, buf ^ 1);  // its last readers passed the previous barrier
        __syncthreads();
    }
}

template <int DK, int OPT, int NS>
hipError_t launch_tree_ns(const ScanTreeParams& p, long nb, hipStream_t s, const GdnArgs& a) {
    using T = typename Op<OPT>::T;
    hipLaunchKernelGGL((scan_tree_kernel<DK, OPT, NS>), dim3((unsigned)nb), dim3(256), 0, s, p, static_cast<const T*>(a.q),
                       static_cast<const T*>(a.k), static_cast<const T*>(a.v), a.g, a.beta, a.state0,
                       static_cast<T*>(a.o));
    return hipGetLastError();
}

constexpr int kScanSlots = 4;  // most saved states (registers) of scan_tree_kernel

template <int OPT>
hipError_t launch_tree(int dk, const ScanTreeParams& p, long nb, hipStream_t s, const GdnArgs& a) {
    switch (dk) {
        case 16: return launch_tree_ns<16, OPT, kScanSlots>(p, nb, s, a);
        case 32: return launch_tree_ns<32, OPT, kScanSlots>(p, nb, s, a);
        case 64: return launch_tree_ns<64, OPT, kScanSlots>(p, nb, s, a);
        default: return launch_tree_ns<128, OPT, kScanSlots>(p, nb, s, a);
    }
}

// Whether scan_tree_kernel takes a call: plans that carry the traversal and need at most
// kScanSlots saved states, without node-state dump or operand preparation, where it is the
// faster form (8 requests x 6 layers x 64 nodes, 32 heads, d = 128: 1,175 -> 280 us; small
// calls with wide trees, and trees of a few nodes, are not: scan_tree_faster).
bool scan_tree_takes(const lumo_gdn_dims& d, const lumo_tree_desc& desc, const GdnArgs& a, int64_t section) {
    if (section < 0 || desc.host_blob[section] > kScanSlots || a.node_states || a.prep.flags != 0) return false;
    return scan_tree_faster(d, desc.plan, desc.host_blob);
}

template <int DK, int OPT>
void launch_one(dim3 grid, hipStream_t s, const ScanParams& p, const GdnArgs& a) {
    using T = typename Op<OPT>::T;
    hipLaunchKernelGGL((scan_kernel<DK, OPT>), grid, dim3(64), 0, s, p, static_cast<const T*>(a.q),
                       static_cast<const T*>(a.k), static_cast<const T*>(a.v), a.g, a.beta, a.state0,
                       static_cast<T*>(a.o), a.node_states, a.ws);
}

template <int OPT>
hipError_t launch_dk(int dk, dim3 grid, hipStream_t s, const ScanParams& p, const GdnArgs& a) {
    switch (dk) {
        case 16: launch_one<16, OPT>(grid, s, p, a); break;
        case 32: launch_one<32, OPT>(grid, s, p, a); break;
        case 64: launch_one<64, OPT>(grid, s, p, a); break;
        default: launch_one<128, OPT>(grid, s, p, a); break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_scan(const lumo_gdn_dims& d, const lumo_tree_desc& desc, const GdnArgs& a, hipStream_t s) {
    const lumo_plan& pl = desc.plan;
    const int64_t section = scan_section(pl, desc.host_blob);
    if (scan_tree_takes(d, desc, a, section)) {
        ScanTreeParams p;
        p.blob = desc.blob;
        p.o_node_off = pl.o_node_off;
        p.o_order = (int32_t)section + kScanHead;
        p.n_layers = d.n_layers;
        p.total_rows = pl.total_rows;
        p.h_k = d.h_k;
        p.h_v = d.h_v;
        p.d_v = d.d_v;
        p.group = d.h_v / d.h_k;
        p.n_ct = d.d_v / 16;
        p.nwk = p.group * p.n_ct;
        p.n_wb = (p.nwk + 3) / 4;
        const long nb = (long)d.n_req * d.n_layers * d.h_k * p.n_wb;
        return d.op_dtype == LUMO_BF16 ? launch_tree<1>(d.d_k, p, nb, s, a) : launch_tree<0>(d.d_k, p, nb, s, a);
    }
    ScanParams p;
    p.blob = desc.blob;
    p.o_seg = pl.o_seg;
    p.o_seg_nodes = pl.o_seg_nodes;
    p.n_layers = d.n_layers;
    p.total_rows = pl.total_rows;
    p.h_k = d.h_k;
    p.h_v = d.h_v;
    p.d_v = d.d_v;
    p.group = d.h_v / d.h_k;
    p.n_vtiles = (d.d_v + 63) / 64;
    p.prep = a.prep;
    // Level boundaries come from the host copy of the plan words.
    for (int lv = 0; lv < pl.n_levels; ++lv) {
        const int first = desc.host_blob[pl.o_level_off + lv];
        const int count = desc.host_blob[pl.o_level_off + lv + 1] - first;
        if (count <= 0) continue;
        p.seg_first = first;
        const long blocks = (long)count * d.n_layers * d.h_v * p.n_vtiles;
        hipError_t e = d.op_dtype == LUMO_BF16 ? launch_dk<1>(d.d_k, dim3((unsigned)blocks), s, p, a)
                                               : launch_dk<0>(d.d_k, dim3((unsigned)blocks), s, p, a);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lumo
