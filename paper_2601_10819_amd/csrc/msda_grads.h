// The backward gather's unit of work, shared by every work order: the
// gradients of a run of one anchor's (keypoint, camera) pairs, by one wave.
//
// What bounds it: at the 64-camera scene in BF16 the vector ALU is busy 86% of
// the launch (61 instructions per sample: 32 widen and multiply-add the
// corners, 12 form the sums, the rest stages and reduces) and the vector
// cache's address path 92%. One camera per unit keeps an XCD's waves on one
// camera's pyramid, each sample is staged by one lane with its record, and
// grad_w leaves by whole samples: 0.44 -> 0.39 ms. Products on the matrix
// cores (grad_out split exactly into three bfloat16 parts, the diagonal of
// 4x4x4 blocks) took the vector ALU to 50 instructions per sample and not
// the time: 0.40 ms.
//
// Per sample it re-gathers the 4 corners and forms d[c] = <grad_out, corner c>
// over the lane's channels; grad_w is a sum over the group's lanes of the
// corner weights times d, grad_loc one over the sample's lanes, once per pair,
// of the blend's derivatives times the weights. The lane that stages a sample
// also writes its grad_feat record.
#pragma once

#include "msda_common.h"

namespace msda {

// Staging: one sample per lane, lane = pair * Lp + level with the levels
// padded to a power of two, so grad_samples / Lp pairs at a time. With 64 groups
// half a wave's lanes, whose LDS leaves room for 16 waves per CU instead of 8
// (16 cameras of 256 x 448, 900 anchors, FP32: 376 -> 264 us). Per sample in LDS:
// corner offsets, corner weights, location-derivative factors (W(1-ly), W ly,
// H(1-lx), H lx), and its G weights, which its grad_w replaces.
__host__ __device__ constexpr int level_shift(int L) {
    return L > 4 ? 3 : L > 2 ? 2 : L > 1 ? 1 : 0;
}
__host__ __device__ constexpr int grad_samples(int G) { return G > 32 ? 32 : 64; }
// (of a PACKED kernel, with no more than kPackedGroups groups: a constant)
template <bool PACKED>
__host__ __device__ constexpr int grad_samples_of(int G) { return PACKED ? 64 : grad_samples(G); }
__host__ __device__ constexpr size_t grads_lds_bytes(int G) {
    return (size_t)grad_samples(G) * (3 * 16 + 4 * (size_t)G + 4);
}

struct GradLds {
    u32x4* off;
    float4* cw;
    float4* dk;
    float* w;
    u32* src;                // per pair: its index p*N + n among the anchor's pairs
};

template <bool PACKED>
__device__ __forceinline__ GradLds grads_lds(unsigned char* p, int G) {
    const int n = grad_samples_of<PACKED>(G);
    GradLds s;
    s.off = reinterpret_cast<u32x4*>(p);
    s.cw = reinterpret_cast<float4*>(s.off + n);
    s.dk = s.cw + n;
    s.w = reinterpret_cast<float*>(s.dk + n);
    s.src = reinterpret_cast<u32*>(s.w + n * G);
    return s;
}

// Where the samples' grad_feat records go. The sample (pair src, level l) has
// the index s = base + src*L + l; its fractions go to frac[s]. Bucketed
// records (ap != 0): to bucket (b, n, l) at slot a*P + p, i.e.
// key[bucket_base + (n*L + l)*ap + p], the key the local cell of the region
// ((H+1)(W+1) outside the level). Compacted records (val != nullptr, the
// visible-view form with the global sort): the k-th pair's record is r =
// cbase + k*L + l, key[r] the cell and val[r] = s. Else key[s] = the cell.
struct RecordSink {
    u32* key;                // nullptr: no records
    float2* frac;
    u32 base;                // first sample of the anchor
    u32 cell_base;           // first cell of the batch item
    u32 no_cell;             // key of a sample outside its level
    u32* val;
    u32 cbase;
    u32 ap;                  // bucketed: records per bucket (0: not bucketed)
    u32 bucket_base;         // bucketed: b*N*L*A*P + a*P
};

// Per-anchor context of the backward gather.
struct GradAnchor {
    const float* gw;         // weights of the anchor [P*N][L*G]
    const float* gl;         // locations [P*N][2]
    const float* go;         // grad_out row
    float* gwout;            // grad_weights of the anchor (or nullptr)
    float* glout;            // grad_sampling_loc of the anchor (or nullptr)
    float* gacc;             // atomic grad_feat: FP32 accumulator of the batch item (or nullptr)
    RecordSink rec;
    rsrc_t feat;
};

template <class FT>
__device__ __forceinline__ GradAnchor grad_anchor(const OpArgs& a, int b, int an) {
    const size_t ba = (size_t)b * a.A + an;
    const size_t npairs = (size_t)a.P * a.N, LG = (size_t)a.L * a.G;
    GradAnchor x;
    x.gw = a.w + ba * npairs * LG;
    x.gl = a.loc + ba * npairs * 2;
    x.go = a.grad_out + ba * a.C;
    x.gwout = a.grad_w ? a.grad_w + ba * npairs * LG : nullptr;
    x.glout = a.grad_loc ? a.grad_loc + ba * npairs * 2 : nullptr;
    x.gacc = a.gfeat_acc ? a.gfeat_acc + (size_t)b * a.R * a.C : nullptr;
    x.rec.key = a.rec_key;
    x.rec.frac = a.rec_frac;
    x.rec.base = a.sample_offset + (u32)ba * (u32)npairs * (u32)a.L;
    x.rec.cell_base = a.cell_offset + (u32)b * a.cells_per_item;
    x.rec.no_cell = a.no_cell;
    x.rec.val = nullptr;
    x.rec.cbase = 0u;
    x.rec.ap = a.rec_bucket_ap;
    x.rec.bucket_base = a.sample_offset + (u32)b * (u32)(a.N * a.L) * a.rec_bucket_ap +
                        (u32)an * (u32)a.P;
    x.feat = make_rsrc(static_cast<const char*>(a.feat) + (size_t)b * a.batch_bytes,
                       a.batch_bytes);
    return x;
}

// Pair orders: the k-th pair -> keypoint p, camera n. Both walk the cameras one
// after the other: anchor order's wave all of the anchor's, taking every
// nwaves-th pair, view order's those from n_lo on.
struct AnchorOrder {
    int P, nwaves, wave;
    u32 m;                   // div_magic(P, pairs)
    __device__ __forceinline__ void operator()(int k, int* p, int* n) const {
        const int i = k * nwaves + wave;
        *n = div_by(i, P, m);
        *p = i - *n * P;
    }
};

struct ViewOrder {
    int P, n_lo;
    u32 m;                   // div_magic(P, pairs)
    __device__ __forceinline__ void operator()(int k, int* p, int* n) const {
        const int q = div_by(k, P, m);
        *p = k - q * P;
        *n = n_lo + q;
    }
};

// Stages pairs [k0, k0 + nj) and writes their records; lanes past the last
// sample stage zeros that read no memory.
template <class FT, bool PACKED, class Order>
__device__ __forceinline__ void stage_grads(const OpArgs& a, const GradAnchor& x,
                                            const Order& order, int k0, int nj, int lane,
                                            const GradLds& s) {
    const int L = a.L, G = a.G, ls = level_shift(L);
    const int jj = lane >> ls, l = lane & ((1 << ls) - 1);
    u32x4 off = {kOOB, kOOB, kOOB, kOOB};
    float4 cw = make_float4(0.f, 0.f, 0.f, 0.f), dk = cw;
    const bool live = jj < nj && l < L;
    u32 row = 0;                                    // the sample's row of G weights
    if (live) {
        int p, n;
        order(k0 + jj, &p, &n);
        const u32 src = (u32)p * (u32)a.N + (u32)n;
        const int r = n * L + l;
        Geo gm = {};
        gm.H = a.shapes[2 * r];
        gm.W = a.shapes[2 * r + 1];
        gm.start = a.starts[r];
        row = src * (u32)L + (u32)l;
        const Corners c = corners_of(x.gl[2 * (size_t)src], x.gl[2 * (size_t)src + 1], gm,
                                     (u32)a.C * FT::kBytes, 0u);
        off = u32x4{c.off[0], c.off[1], c.off[2], c.off[3]};
        cw = make_float4(c.cw[0], c.cw[1], c.cw[2], c.cw[3]);
        const float fw = (float)gm.W, fh = (float)gm.H;
        dk = make_float4(fw * (1.f - c.ly), fw * c.ly, fh * (1.f - c.lx), fh * c.lx);
        if (l == 0) s.src[jj] = src;
        if (x.rec.key) {
            const u32 smp = x.rec.base + src * (u32)L + (u32)l;
            const u32 local = c.valid ? (u32)(c.y0 + 1) * (u32)(gm.W + 1) + (u32)(c.x0 + 1)
                                      : (u32)(gm.H + 1) * (u32)(gm.W + 1);
            if (x.rec.ap) {
                x.rec.key[x.rec.bucket_base + (u32)r * x.rec.ap + (u32)p] = local;
            } else {
                const u32 key = c.valid ? x.rec.cell_base + a.cell_start[r] + local
                                        : x.rec.no_cell;
                u32 at = smp;
                if (x.rec.val) {
                    at = x.rec.cbase + (u32)(k0 + jj) * (u32)L + (u32)l;
                    x.rec.val[at] = smp;
                }
                x.rec.key[at] = key;
            }
            x.rec.frac[smp] = make_float2(c.lx, c.ly);
        }
    }
    const int ns = grad_samples_of<PACKED>(G);
    if (lane < ns) {
        s.off[lane] = off;
        s.cw[lane] = cw;
        s.dk[lane] = dk;
    }
    if constexpr (!PACKED) {
        // lane after lane across a sample's groups (64 % G == 0): the loads and LDS
        // stores of a lane's own sample would be G entries apart in the wave
        const u32 r = live ? row : ~0u;
        const int gs = __builtin_ctz(G), g = lane & (G - 1);
        for (int e0 = lane; e0 - lane < ns * G; e0 += 64 * 8) {      // ns * G >= 1024
            float t[8];
            bool in[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const u32 i = (u32)__shfl((int)r, (e0 + 64 * k) >> gs, 64);
                in[k] = i != ~0u;
                t[k] = x.gw[(size_t)(in[k] ? i : 0u) * (u32)G + (u32)g];
            }
#pragma unroll
            for (int k = 0; k < 8; ++k) s.w[e0 + 64 * k] = in[k] ? t[k] : 0.f;
        }
    } else if (G == 8) {
        const float* w = x.gw + (size_t)row * (u32)G;
        float t[8];
#pragma unroll
        for (int g = 0; g < 8; ++g) t[g] = live ? w[g] : 0.f;
        float4* d = reinterpret_cast<float4*>(s.w + lane * 8);
        d[0] = make_float4(t[0], t[1], t[2], t[3]);
        d[1] = make_float4(t[4], t[5], t[6], t[7]);
    } else {
        const float* w = x.gw + (size_t)row * (u32)G;
        for (int g = 0; g < G; ++g) s.w[lane * G + g] = live ? w[g] : 0.f;
    }
}

// Levels of a pair whose corner loads are issued together. At the 64-camera
// scene in BF16: 2 levels 0.391 ms (73 VGPRs), 4 0.413 (110).
constexpr int kGradLevels = 2;

// The gradients of the staged pairs: grad_w of their samples into s.w,
// grad_loc to memory. out_scale multiplies both (the fused form's per-view
// weight); dot (or nullptr) accumulates, on each group's first lane,
// <grad_out, the pairs' feature>.
template <class FT, int CPL, bool PACKED, int LPG, int LPS>
__device__ __forceinline__ void pairs_grads(const OpArgs& a, const GradAnchor& x, const GradLds& s,
                                            int nj, const Lanes& q, const float* go,
                                            float out_scale, float* dot) {
    using RowT = Row<FT, CPL>;
    constexpr int LU = kGradLevels;
    const int L = a.L, G = a.G, ls = level_shift(L), J = grad_samples_of<PACKED>(G) >> ls;
    const int lpg = (a.C / G) / CPL;               // lanes of one group (a power of two)
    for (int j0 = 0; j0 < nj; j0 += q.spw) {
        // sub-waves past the last pair repeat one and write nothing
        const int jj = j0 + q.sub, e = min(jj, J - 1);
        const bool ok = jj < nj;
        float gx = 0.f, gy = 0.f;
        for (int l0 = 0; l0 < L; l0 += LU) {
            u32 raw[LU][4][RowT::kWords];
#pragma unroll
            for (int k = 0; k < LU; ++k) {
                // levels past L read nothing
                const u32x4 o = s.off[(e << ls) + min(l0 + k, L - 1)];
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    load_words<RowT::kWords>(x.feat, l0 + k < L ? o[c] + q.lane_off : kOOB,
                                             raw[k][c]);
            }
            // the compiler would sink each load to its use and wait for every pair
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < LU; ++k) {
                const int l = l0 + k;
                if (l >= L) break;
                float d[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float f[CPL];
                    widen<FT, CPL>(raw[k][c], f);
                    float sum = 0.f;
#pragma unroll
                    for (int i = 0; i < CPL; ++i) sum = fmaf(go[i], f[i], sum);
                    d[c] = sum;
                }
                const int i = (e << ls) + l;
                const float4 cw = s.cw[i], dk = s.dk[i];
                float* wp = s.w + i * G + q.g;
                const float wl = *wp;
                float tw = cw.x * d[0] + cw.y * d[1] + cw.z * d[2] + cw.w * d[3];
                tw = group_sum_w<LPG>(tw, lpg);
                if (ok && (q.lane & (lpg - 1)) == 0) {
                    *wp = tw * out_scale;
                    if (dot) *dot = fmaf(wl, tw, *dot);
                }
                // d val / dx = W ((1-ly)(F01 - F00) + ly (F11 - F10)) (x = u W - 0.5),
                // and d val / dy alike, the factors staged per sample
                gx = fmaf(wl, dk.x * (d[1] - d[0]) + dk.y * (d[3] - d[2]), gx);
                gy = fmaf(wl, dk.z * (d[2] - d[0]) + dk.w * (d[3] - d[1]), gy);
            }
        }
        if (x.glout) {
            gx = group_sum_w<LPS>(gx, q.lps);
            gy = group_sum_w<LPS>(gy, q.lps);
            if (ok && (q.lane & (q.lps - 1)) == 0) {
                const size_t src = s.src[jj];
                x.glout[src * 2] = gx * out_scale;
                x.glout[src * 2 + 1] = gy * out_scale;
            }
        }
    }
}

// Adds w * cw * grad_out of the staged pairs' corners into the FP32
// accumulator with float atomics (the atomic grad_feat form).
template <class FT, int CPL>
__device__ __forceinline__ void pairs_atomic(const OpArgs& a, const GradAnchor& x,
                                             const GradLds& s, int nj, const Lanes& q) {
    // byte offset of a row -> float offset in the FP32 accumulator
    constexpr int kOffToAcc = FT::kBytes == 4 ? 2 : FT::kBytes == 2 ? 1 : 0;
    const int ls = level_shift(a.L);
    float go[CPL];
#pragma unroll
    for (int i = 0; i < CPL; ++i) go[i] = x.go[q.c0 + i];
    for (int jj = q.sub; jj < nj; jj += q.spw) {
        for (int l = 0; l < a.L; ++l) {
            const int i = (jj << ls) + l;
            const u32x4 off = s.off[i];
            const float4 c4 = s.cw[i];
            const float cw[4] = {c4.x, c4.y, c4.z, c4.w};
            const float wl = s.w[i * a.G + q.g];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (off[c] != kOOB) {
                    float* dst = x.gacc + q.c0 + (off[c] >> kOffToAcc);
                    const float cwl = cw[c] * wl;
#pragma unroll
                    for (int k = 0; k < CPL; ++k) unsafeAtomicAdd(dst + k, cwl * go[k]);
                }
            }
        }
    }
}

// The gradients and records of pairs [k_lo, k_hi) (in the order's numbering).
// The lane widths of the common layouts (C = 256 in G = 8 groups: 32 lanes
// per sample in groups of 4 with 8 channels per lane, 64 in groups of 8 with
// 4) are compile-time in their copies of the loop.
template <class FT, int CPL, bool PACKED, class Order>
__device__ __forceinline__ void grads_of(const OpArgs& a, const GradAnchor& x, const Order& order,
                                         int k_lo, int k_hi, const Lanes& q, unsigned char* lds,
                                         float out_scale = 1.f, float* dot = nullptr) {
    const GradLds s = grads_lds<PACKED>(lds, a.G);
    const int G = a.G, L = a.L, ls = level_shift(L), J = grad_samples_of<PACKED>(G) >> ls;
    const int lpg = (a.C / G) / CPL;
    float go[CPL];
#pragma unroll
    for (int i = 0; i < CPL; ++i) go[i] = x.go[q.c0 + i];
    for (int k0 = k_lo; k0 < k_hi; k0 += J) {
        const int nj = min(J, k_hi - k0);
        stage_grads<FT, PACKED>(a, x, order, k0, nj, q.lane, s);
        wave_lds_sync();
        if (x.gacc) pairs_atomic<FT, CPL>(a, x, s, nj, q);
        if (x.gwout || x.glout || dot) {
            if (PACKED && lpg == 4 && q.lps == 32)
                pairs_grads<FT, CPL, PACKED, 4, 32>(a, x, s, nj, q, go, out_scale, dot);
            else if (PACKED && lpg == 8 && q.lps == 64)
                pairs_grads<FT, CPL, PACKED, 8, 64>(a, x, s, nj, q, go, out_scale, dot);
            else
                pairs_grads<FT, CPL, PACKED, 0, 0>(a, x, s, nj, q, go, out_scale, dot);
            wave_lds_sync();
            // grad_w, a sample's groups by the lane that staged it, or (many) lane
            // after lane
            const int jj = q.lane >> ls, l = q.lane & ((1 << ls) - 1);
            if (!PACKED && x.gwout) {
                const int gs = __builtin_ctz(G);
                for (int e = q.lane; e < grad_samples(G) * G; e += 64) {
                    const int je = e >> gs >> ls, le = (e >> gs) & ((1 << ls) - 1);
                    if (je < nj && le < L)
                        x.gwout[((size_t)s.src[je] * L + le) * G + (e & (G - 1))] = s.w[e];
                }
            } else if (x.gwout && jj < nj && l < L) {
                float* o = x.gwout + ((size_t)s.src[jj] * L + l) * G;
                const float* t = s.w + q.lane * G;
                if (G == 8) {
#pragma unroll
                    for (int g = 0; g < 8; ++g) o[g] = t[g];
                } else {
                    for (int g = 0; g < G; ++g) o[g] = t[g];
                }
            }
        }
        wave_lds_sync();
    }
}

}  // namespace msda
