// The forwards' unit of work: a run of one anchor's samples, by one wave.
// Shared by every work order.
//
// What bounds it: the corner rows' path through the vector cache. At the
// 64-camera scene in BF16 a kernel that only loads the same rows takes 0.28
// ms of this one's 0.32 (21 TB/s; rows that stay in one XCD's 4 MB L2 come at
// 29 TB/s). So in view order the units run camera by camera -- an XCD's waves work on one
// camera's pyramid at a time -- and the work around the loads is kept off the
// waves' critical path: 16 corner loads in flight per wave, the corner
// weights multiplied out once per sample and group while staging, no
// block-wide step. Before, a wave took an anchor through all of its XCD's
// cameras and the multiply-adds waited for their loads two by two: 0.385 ms
// in BF16 (0.325 now), 0.727 in FP32 (0.577), 0.345 in FP8 (0.230).
#pragma once

#include "msda_common.h"

namespace msda {

// Rounds of samples whose corner loads are issued together.
constexpr int kRowRounds = 4;

// A wave's staged samples: corner offsets, corner weights (PACKED: per group,
// times the group's weight) and the groups' weights (not PACKED). PACKED is the
// kernel's own: both walks in one took the FP8 kernel from 126 to 153 registers
// (0.23 -> 0.27 ms at the 64-camera scene).
struct RowLds {
    u32x4* off;
    float4* cw;
    float* w;
};

__device__ __forceinline__ RowLds row_lds(unsigned char* p, int chunk) {
    RowLds s;
    s.off = reinterpret_cast<u32x4*>(p);
    s.cw = reinterpret_cast<float4*>(s.off + chunk);
    s.w = reinterpret_cast<float*>(s.cw + chunk);
    return s;
}

// U rounds of staged samples from round t (64 / lanes-per-sample samples
// each): the corner loads of all U, then their multiply-adds.
template <class FT, int CPL, bool PACKED, int U>
__device__ __forceinline__ void row_rounds(const Lanes& q, rsrc_t feat, int t, int G,
                                           const RowLds& s, float* acc) {
    using RowT = Row<FT, CPL>;
    u32 raw[U][4][RowT::kWords];
#pragma unroll
    for (int x = 0; x < U; ++x) {
        const u32x4 o = s.off[(t + x) * q.spw + q.sub];
#pragma unroll
        for (int c = 0; c < 4; ++c) load_words<RowT::kWords>(feat, o[c] + q.lane_off, raw[x][c]);
    }
    // the compiler would sink each load to its use and wait for every pair
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int x = 0; x < U; ++x) {
        const int i = (t + x) * q.spw + q.sub;
        float4 w = s.cw[PACKED ? i * G + q.g : i];
        if constexpr (!PACKED) {
            const float wg = s.w[i * G + q.g];
            w = make_float4(w.x * wg, w.y * wg, w.z * wg, w.w * wg);
        }
        const float wc[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float f[CPL];
            widen<FT, CPL>(raw[x][c], f);
#pragma unroll
            for (int i = 0; i < CPL; ++i) acc[i] = fmaf(wc[c], f[i], acc[i]);
        }
    }
}

// All rounds of the ns staged samples.
template <class FT, int CPL, bool PACKED>
__device__ __forceinline__ void row_walk(const Lanes& q, rsrc_t feat, int ns, int G,
                                         const RowLds& s, float* acc) {
    const int rounds = (ns + q.spw - 1) / q.spw;
    int t = 0;
    for (; t + kRowRounds <= rounds; t += kRowRounds)
        row_rounds<FT, CPL, PACKED, kRowRounds>(q, feat, t, G, s, acc);
    if (t + 2 <= rounds) {
        row_rounds<FT, CPL, PACKED, 2>(q, feat, t, G, s, acc);
        t += 2;
    }
    if (t < rounds) row_rounds<FT, CPL, PACKED, 1>(q, feat, t, G, s, acc);
}

// The weights of the first entries / G staged samples, more than kPackedGroups
// groups each, lane after lane across a sample's groups: `row` is this lane's
// sample's row of G weights among the anchor's (0 past the ns-th sample, whose
// weights become 0). A lane taking its own sample's would leave every load and
// LDS store of the wave G entries apart.
__device__ __forceinline__ void stage_weights(const WSrc& gw, u32 row, int ns, int G, int entries,
                                              int lane, float* s_w) {
    constexpr int U = 8;
    const int gs = __builtin_ctz(G), g = lane & (G - 1);      // 64 % G == 0
    const float2 st = gw.stats ? gw.stats[g] : make_float2(0.f, 0.f);
    for (int e0 = lane; e0 - lane < entries; e0 += 64 * U) {
        float v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int i = (e0 + 64 * k) >> gs;
            v[k] = gw.raw((size_t)(u32)__shfl((int)row, i & 63, 64) * (u32)G + (u32)g);
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int e = e0 + 64 * k;
            const float w = gw.stats ? expf(v[k] - st.x) * st.y : v[k];
            if (e < entries) s_w[e] = e >> gs < ns ? w : 0.f;
        }
    }
}

// Sums the per-sample partials of a wave's sub-waves (samples that share
// channels): a butterfly over the sub-wave index.
template <int CPL>
__device__ __forceinline__ void reduce_subwaves(const Lanes& q, float* acc) {
    for (int s = q.lps; s < 64; s <<= 1) {
#pragma unroll
        for (int i = 0; i < CPL; ++i) acc[i] = xor_sum(acc[i], s);
    }
}

// The sum of samples [s_lo, s_hi) of anchor `ba` over the lane's channels, the
// same in every sub-wave. The anchor's samples are numbered camera-major,
// then keypoint, then level; they go through LDS `chunk` at a time (a power of two from
// the sub-waves' count to 64; it does not change the sum's order), one per
// lane: corner offsets, and per group the corner weights times the sample's
// weight (and the FP8 level scale; many groups: apart, see row_lds_bytes).
// Geometry is read from memory: a camera's few words stay in the caches, and
// nothing is staged block-wide.
template <class FT, int CPL, bool PACKED>
__device__ __forceinline__ void row_sum(const OpArgs& a, size_t ba, rsrc_t feat, int s_lo,
                                        int s_hi, const Lanes& q, int chunk, unsigned char* lds,
                                        float* acc) {
    const int L = a.L, G = a.G, P = a.P, LG = L * G, npairs = P * a.N;
    const float* gl = a.loc + ba * npairs * 2;
    const WSrc gw = anchor_weights(a, ba, (size_t)npairs * LG);
    const u32 row_bytes = (u32)a.C * FT::kBytes;
    const int NS = P * L;
    const u32 mL = div_magic(L, NS), mNS = div_magic(NS, s_hi);
    const RowLds rl = row_lds(lds, chunk);
#pragma unroll
    for (int i = 0; i < CPL; ++i) acc[i] = 0.f;
    for (int i0 = s_lo; i0 < s_hi; i0 += chunk) {
        const int i = i0 + q.lane, ns = min(chunk, s_hi - i0);
        // lanes past the last sample stage zeros that read no memory
        const bool live = q.lane < ns;
        u32x4 off = {kOOB, kOOB, kOOB, kOOB};
        float4 cw = make_float4(0.f, 0.f, 0.f, 0.f);
        size_t wb = 0;
        u32 row = 0;
        if (live) {
            const int n = div_by(i, NS, mNS), k = i - n * NS;
            const int p = div_by(k, L, mL), l = k - p * L;
            const size_t src = (size_t)p * a.N + n;
            const int r = n * L + l;
            Geo gm = {};
            gm.H = a.shapes[2 * r];
            gm.W = a.shapes[2 * r + 1];
            gm.start = a.starts[r];
            wb = src * LG + (size_t)(l * G);
            row = (u32)src * (u32)L + (u32)l;
            const Corners c = corners_of(gl[2 * src], gl[2 * src + 1], gm, row_bytes, 0u);
            off = u32x4{c.off[0], c.off[1], c.off[2], c.off[3]};
            const float s = FT::kBytes == 1 ? a.level_scale[l] : 1.f;
            cw = FT::kBytes == 1 ? make_float4(c.cw[0] * s, c.cw[1] * s, c.cw[2] * s, c.cw[3] * s)
                                 : make_float4(c.cw[0], c.cw[1], c.cw[2], c.cw[3]);
        }
        auto put = [&](int g, float w) {
            rl.cw[q.lane * G + g] = make_float4(cw.x * w, cw.y * w, cw.z * w, cw.w * w);
        };
        if (q.lane < chunk) {
            rl.off[q.lane] = off;
            if constexpr (!PACKED) {
                rl.cw[q.lane] = cw;
            } else if (G == 8) {
                float w[8];
#pragma unroll
                for (int g = 0; g < 8; ++g) w[g] = live ? gw.raw(wb + g) : 0.f;
                if (gw.stats && live) {
#pragma unroll
                    for (int g = 0; g < 8; ++g) w[g] = gw.softmax(w[g], g);
                }
#pragma unroll
                for (int g = 0; g < 8; ++g) put(g, w[g]);
            } else {
                for (int g = 0; g < G; ++g) {
                    float w = live ? gw.raw(wb + g) : 0.f;
                    if (gw.stats && live) w = gw.softmax(w, g);
                    put(g, w);
                }
            }
        }
        if constexpr (!PACKED)
            stage_weights(gw, row, ns, G, (ns + q.spw - 1) / q.spw * q.spw * G, q.lane, rl.w);
        wave_lds_sync();
        row_walk<FT, CPL, PACKED>(q, feat, ns, G, rl, acc);
        wave_lds_sync();
    }
    reduce_subwaves<CPL>(q, acc);
}

}  // namespace msda
