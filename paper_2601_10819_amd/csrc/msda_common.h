// Device-side building blocks shared by the MSDA kernels for gfx950:
// buffer resources and lane-width loads, storage widening, sample geometry,
// and the per-wave LDS staging of locations and weights.
//
// The operator (paper Sec. 3.1 / Sec. 3.2; named in Sec. 5.3) samples every
// camera's feature pyramid bilinearly at each projected keypoint and sums the
// samples with per-(keypoint, camera, level, group) weights. It is a gather
// with low arithmetic intensity (Sec. 5.3), so the kernels are organised
// around memory access, not matrix cores:
//
//  * Each lane owns CPL consecutive channels; a sample occupies C/CPL lanes
//    ("lanes per sample", a power of two <= 64) and a 64-lane wave works on
//    64/(C/CPL) samples at once. Corner rows are read with 4/8/16-byte buffer
//    loads, so the 4 corner gathers of a sample are channel-contiguous.
//  * Feature reads go through a buffer resource spanning one batch item. A
//    corner outside its level gets an offset past the end of the resource and
//    the hardware returns 0 without touching memory: zero padding costs no
//    branch, and no computed index can read outside the tensor.
//  * The coordinate t = u*W - 0.5 is assembled from the exact product u*W
//    (an fma recovers the rounding error of the multiply), so floor(t) and the
//    bilinear fraction are exact to ~1e-7 px instead of half an FP32 ulp of t.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "msda_internal.h"

namespace msda {

typedef uint32_t u32;
typedef uint64_t u64;
typedef u32 u32x2 __attribute__((ext_vector_type(2)));
typedef u32 u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;


// Word 3 of a raw (untyped, stride 0) buffer resource on gfx9-family GPUs.
constexpr int kRsrcWord3 = 0x00020000;

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, u32 bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                             kRsrcWord3);
}

// ---------------------------------------------------------------- storage types

// kKind matches the FeatType code of the storage type.
struct TF32 { static constexpr int kBytes = 4, kKind = 0; };
struct TBF16 { static constexpr int kBytes = 2, kKind = 1; };
struct TFP8 { static constexpr int kBytes = 1, kKind = 2; };
struct TF16 { static constexpr int kBytes = 2, kKind = 3; };

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

template <class FT, int CPL>
struct Row {
    static constexpr int kBytes = FT::kBytes * CPL;   // 4, 8 or 16
    static constexpr int kWords = kBytes / 4;
    static_assert(kBytes == 4 || kBytes == 8 || kBytes == 16, "unsupported lane width");
};

template <int WORDS>
__device__ __forceinline__ void load_words(rsrc_t r, u32 off, u32* d) {
    if constexpr (WORDS == 4) {
        u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
    } else if constexpr (WORDS == 2) {
        u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        d[0] = v.x; d[1] = v.y;
    } else {
        d[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
    }
}

// Widen CPL stored channels (packed in `w`) to FP32.
template <class FT, int CPL>
__device__ __forceinline__ void widen(const u32* w, float* f) {
    if constexpr (FT::kBytes == 4) {
#pragma unroll
        for (int i = 0; i < CPL; ++i) f[i] = __uint_as_float(w[i]);
    } else if constexpr (FT::kKind == 1) {
        // bfloat16 is the top half of an FP32: widening is a shift.
#pragma unroll
        for (int i = 0; i < CPL / 2; ++i) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    } else if constexpr (FT::kKind == 3) {
        // IEEE half to FP32 is exact; feeding it straight into an FMA lets the
        // compiler use v_fma_mix_f32, which widens either half of a word
        // inside the FP32 FMA itself.
#pragma unroll
        for (int i = 0; i < CPL / 2; ++i) {
            const half2_t h = __builtin_bit_cast(half2_t, w[i]);
            f[2 * i] = (float)h.x;
            f[2 * i + 1] = (float)h.y;
        }
    } else {
        // OCP e4m3 to FP32 with the hardware converter, two codes at a time.
#pragma unroll
        for (int i = 0; i < CPL / 4; ++i) {
            f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[i], false);
            f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[i], true);
            f[4 * i] = lo.x; f[4 * i + 1] = lo.y; f[4 * i + 2] = hi.x; f[4 * i + 3] = hi.y;
        }
    }
}

// FP32 -> IEEE half with the hardware conversion: round to nearest even
// (the default rounding mode), overflow to infinity, NaN stays NaN.
__device__ __forceinline__ uint16_t f16_rne(float x) {
    return __builtin_bit_cast(uint16_t, (_Float16)x);
}

// FP32 -> bfloat16 with gfx950's converter (v_cvt_pk_bf16_f32): round to
// nearest even, overflow to infinity, NaN stays NaN.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint16_t bf16_rne(float x) {
    return __builtin_bit_cast(uint16_t, (__bf16)x);
}

// Two values at once, lo in the low half: one instruction.
__device__ __forceinline__ u32 bf16x2_rne(float lo, float hi) {
    const bf16x2_t v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(u32, v);
}

// ---------------------------------------------------------------- geometry

// One (camera, level) region: its size and first row.
struct Geo { int H, W, start; };

// Integer part and fraction of t = u*n - 0.5 along one axis of a level with n
// pixels, and whether -1 < t < n. u*n is split exactly into p + e, the floor
// is taken of p, and the fraction is assembled from exact pieces, so only the
// final add rounds.
struct Axis { int i0; float l; bool ok; };

__device__ __forceinline__ Axis axis_of(float u, int n) {
    // The split only works if each operation is rounded as written: a fused
    // u*n - fp would already contain e, which is then added a second time.
#pragma clang fp contract(off)
    const float fn = (float)n;
    const float p = u * fn;
    const float e = fmaf(u, fn, -p);            // u*n == p + e exactly
    const float fp = floorf(p);
    const float f = ((p - fp) - 0.5f) + e;      // t - fp, in about [-0.5, 0.5)
    const float flo = f < 0.f ? -1.f : 0.f;
    float l = f - flo;
    float i0f = fp + flo;
    if (l >= 1.f) { l = 0.f; i0f += 1.f; }      // f a hair below 0: t is an integer
    i0f = fminf(fmaxf(i0f, -4.f), fn + 4.f);    // keeps the int conversion defined; NaN -> -4
    Axis a;
    a.i0 = (int)i0f;
    a.ok = (a.i0 >= 0 || (a.i0 == -1 && l > 0.f)) && a.i0 < n;
    a.l = a.ok ? l : 0.f;
    return a;
}

// The 4 corners of one sample, in the order (y0,x0), (y0,x0+1), (y0+1,x0),
// (y0+1,x0+1): byte offsets (kOOB when outside) and bilinear weights (0 when
// outside).
struct Corners {
    u32 off[4];
    float cw[4];
    float lx, ly;
    int x0, y0;     // top-left neighbour (meaningful when valid)
    bool valid;
};

__device__ __forceinline__ Corners corners_of(float u, float v, const Geo& g, u32 row_bytes,
                                              u32 lane_off) {
    const Axis ax = axis_of(u, g.W);
    const Axis ay = axis_of(v, g.H);
    Corners c;
    c.valid = ax.ok && ay.ok;
    c.x0 = ax.i0;
    c.y0 = ay.i0;
    c.lx = c.valid ? ax.l : 0.f;
    c.ly = c.valid ? ay.l : 0.f;
    const float hx = 1.f - c.lx, hy = 1.f - c.ly;
    const bool in_x0 = ax.i0 >= 0, in_x1 = ax.i0 + 1 < g.W;
    const bool in_y0 = ay.i0 >= 0, in_y1 = ay.i0 + 1 < g.H;
    const bool in[4] = {c.valid && in_y0 && in_x0, c.valid && in_y0 && in_x1,
                        c.valid && in_y1 && in_x0, c.valid && in_y1 && in_x1};
    const float wt[4] = {hy * hx, hy * c.lx, c.ly * hx, c.ly * c.lx};
    const int base = g.start + ay.i0 * g.W + ax.i0;
    const int rows[4] = {base, base + 1, base + g.W, base + g.W + 1};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        c.off[k] = in[k] ? (u32)rows[k] * row_bytes + lane_off : kOOB;
        c.cw[k] = in[k] ? wt[k] : 0.f;
    }
    return c;
}

// ---------------------------------------------------------------- lanes and LDS

// Index of the calling wave in its workgroup, as a wave-uniform (scalar)
// value: the compiler cannot see that threadIdx.x / 64 is the same for the
// whole wave, and values derived from it (a batch item's buffer resource, a
// loop bound) would otherwise live in vector registers -- a buffer load
// with a per-lane resource becomes a loop over the distinct resources.
__device__ __forceinline__ int wave_index() {
    return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// A value the caller knows to be the same in every lane, marked as such for
// the compiler (it is then kept in scalar registers).
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ float xor_shuffle(float v, int mask) {
    return __shfl_xor(v, mask, 64);
}

// Cross-lane steps that stay in the VALU (no LDS round trip): DPP row
// permutations and the gfx950 row / half-wave swaps. Callers keep every
// lane of a group active together, so no step reads a disabled lane.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}

// v + v of the lane 16 (resp. 32) away: the swap pairs rows 0-1 and 2-3
// (resp. the two halves); each lane ends with both values of its pair.
__device__ __forceinline__ float swap16_sum(float v) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                    false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

__device__ __forceinline__ float swap32_sum(float v) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                    false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// Sum over aligned groups of `width` lanes (a power of two <= 64, the same in
// every lane): quad butterflies, then row half-mirror and mirror (pairing
// the halves of 8 and of 16 lanes), then the swaps. Every lane of a group
// ends with its group's sum, the same bits in each.
__device__ __forceinline__ float group_sum(float v, int width) {
    if (width > 1) v += dpp<0xB1>(v);     // quad_perm [1,0,3,2]
    if (width > 2) v += dpp<0x4E>(v);     // quad_perm [2,3,0,1]
    if (width > 4) v += dpp<0x141>(v);    // row_half_mirror
    if (width > 8) v += dpp<0x140>(v);    // row_mirror
    if (width > 16) v = swap16_sum(v);
    if (width > 32) v = swap32_sum(v);
    return v;
}

// group_sum with the width known at compile time (no branches); W = 0:
// the width given at run time.
template <int W>
__device__ __forceinline__ float group_sum_w(float v, int width) {
    if constexpr (W == 0) {
        return group_sum(v, width);
    } else {
        if constexpr (W > 1) v += dpp<0xB1>(v);
        if constexpr (W > 2) v += dpp<0x4E>(v);
        if constexpr (W > 4) v += dpp<0x141>(v);
        if constexpr (W > 8) v += dpp<0x140>(v);
        if constexpr (W > 16) v = swap16_sum(v);
        if constexpr (W > 32) v = swap32_sum(v);
        return v;
    }
}

// v + v[lane ^ mask] for a power-of-two mask (the same in every lane).
__device__ __forceinline__ float xor_sum(float v, int mask) {
    if (mask == 32) return swap32_sum(v);
    if (mask == 16) return swap16_sum(v);
    if (mask == 8) return v + dpp<0x128>(v);   // row_ror:8
    return v + xor_shuffle(v, mask);
}

// Quotients of 0 <= i <= i_max by d: by the multiplier of div_magic where that
// is exact (i_max * d < 2^32, d > 1), else (0) by division.
__device__ __forceinline__ u32 div_magic(int d, int64_t i_max) {
    return d > 1 && (u64)i_max * (u32)d >> 32 == 0 ? 0xffffffffu / (u32)d + 1u : 0u;
}

__device__ __forceinline__ int div_by(int i, int d, u32 m) {
    return m ? (int)__umulhi((u32)i, m) : i / d;
}

// Makes this wave's LDS writes visible to its later reads: LDS accesses of
// one wave are performed in program order; the fences keep the compiler
// from moving the reads that follow above the writes.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One anchor's weights as the gathers stage them: FP32 or bfloat16 storage,
// and optionally logits turned into the per-group softmax on the fly
// (w = exp(logit - max_g) / sum_g, the group's statistics precomputed).
struct WSrc {
    const void* p;          // the anchor's [P*N][L*G] weights or logits
    const float2* stats;    // per group (max, 1/sum), or nullptr (plain weights)
    int G;
    bool bf16;
    __device__ WSrc(const void* w, const float2* st, int g, bool b)
        : p(w), stats(st), G(g), bf16(b) {}
    // entry i as stored (FP32, or bfloat16 widened exactly)
    __device__ __forceinline__ float raw(size_t i) const {
        return bf16 ? __uint_as_float((u32)static_cast<const uint16_t*>(p)[i] << 16)
                    : static_cast<const float*>(p)[i];
    }
    // the softmax weight of a logit x of group g (G is a power of two, and
    // entry i of a chunk belongs to group i & (G - 1))
    __device__ __forceinline__ float softmax(float x, int g) const {
        const float2 st = stats[g];
        return expf(x - st.x) * st.y;
    }
};

// The weights of anchor ba (npw = P*N*L*G entries per anchor) as staged.
__device__ __forceinline__ WSrc anchor_weights(const OpArgs& a, size_t ba, size_t npw) {
    const void* p = a.w_bf16 ? static_cast<const void*>(
                                   reinterpret_cast<const uint16_t*>(a.w) + ba * npw)
                             : static_cast<const void*>(a.w + ba * npw);
    return WSrc(p, a.wstats ? a.wstats + ba * (size_t)a.G : nullptr, a.G, a.w_bf16 != 0);
}

// Lane layout of one wave: CPL channels per lane, C/CPL lanes per sample.
struct Lanes {
    int lane, lps, spw, sub, c0, g;
    u32 lane_off;
};

template <class FT, int CPL>
__device__ __forceinline__ Lanes lanes_of(const OpArgs& a) {
    Lanes q;
    q.lane = threadIdx.x & 63;
    q.lps = 1 << a.lps_shift;
    q.spw = 64 >> a.lps_shift;
    q.sub = q.lane >> a.lps_shift;
    q.c0 = (q.lane & (q.lps - 1)) * CPL;
    q.g = q.c0 / (a.C / a.G);
    q.lane_off = (u32)q.c0 * FT::kBytes;
    return q;
}

// Inclusive scan across the 256 threads of a block (4 waves); returns the
// thread's inclusive sum and the block total in *total.
__device__ __forceinline__ u32 block_inclusive_scan(u32 v, u32* lds4, u32* total) {
    const int lane = threadIdx.x & 63, wave = wave_index();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const u32 t = __shfl_up(v, d, 64);
        if (lane >= d) v += t;
    }
    if (lane == 63) lds4[wave] = v;
    __syncthreads();
    u32 before = 0;
    for (int w = 0; w < wave; ++w) before += lds4[w];
    *total = lds4[0] + lds4[1] + lds4[2] + lds4[3];
    __syncthreads();
    return v + before;
}

// Anchor order: launch(first anchor, anchors) over all B*A anchors, a workgroup
// of `waves` waves each.
template <class F>
hipError_t anchor_parts(const OpArgs& a, int waves, F&& launch) {
    const int64_t total = (int64_t)a.B * a.A, part = (int64_t)(kMaxLaunchWaves / (u32)waves);
    for (int64_t at = 0; at < total; at += part) {
        launch((int)at, (unsigned)(total - at < part ? total - at : part));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------- view order

constexpr u64 kNoUnit = ~(u64)0;

// This wave's unit in the range of its workgroup's XCD slot x (the hardware
// hands workgroups to the XCDs round-robin), or kNoUnit.
__device__ __forceinline__ u64 slot_unit(const SlotCuts& cuts, u32 block, int wave, int nwaves) {
    const u32 x = block % kSlots;
    const u64 u = cuts.first[x] + (u64)(block / kSlots) * (u32)nwaves + (u32)wave;
    return u < cuts.end[x] ? u : kNoUnit;
}

// Unit u of a view-order launch as (row, anchor), units row-major: both the
// same across the wave.
struct RowUnit { u32 row; int a; };

__device__ __forceinline__ RowUnit row_unit(u64 u, int A) {
    const u64 r = u >> 32 ? u / (u32)A : (u64)((u32)u / (u32)A);
    RowUnit t;
    t.row = (u32)uniform((int)r);
    t.a = uniform((int)(u - r * (u32)A));
    return t;
}

// Cameras [lo, hi) of row j of `rows`.
struct CamRange { int lo, hi; };

__device__ __forceinline__ CamRange row_cams(int N, int j, int rows) {
    return CamRange{(int)((u64)N * (u32)j / (u32)rows), (int)((u64)N * (u32)(j + 1) / (u32)rows)};
}

// ---------------------------------------------------------------- batched form

// The scene of a batch item index: the last s with start[s] <= item (start
// is a non-decreasing prefix table of S+1 entries).
__device__ __forceinline__ int scene_of(const u32* start, int S, u32 item) {
    int lo = 0, hi = S - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (start[mid] <= item) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// This wave's unit of a batch: its scene and the unit's number in the scene, both
// the same across the wave; scene -1 past the slot's end. A slot's units are
// its ranges of the scenes, one after the other.
struct SceneUnit { int s; u64 u; };

__device__ __forceinline__ SceneUnit scene_unit(const BatchArgs& b, u32 block, int wave,
                                                int nwaves) {
    const u32 x = block % kSlots;
    const u64 i = b.slot_begin + (u64)(block / kSlots) * (u32)nwaves + (u32)wave;
    const u64* start = b.t.slot_start + x * (u32)(b.S + 1);
    if (i >= start[b.S]) return SceneUnit{-1, 0};
    int lo = 0, hi = b.S - 1;                       // the last scene with start <= i
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (start[mid] <= i) lo = mid; else hi = mid - 1;
    }
    const int s = uniform(lo);
    return SceneUnit{s, b.t.slot_first[x * (u32)b.S + (u32)s] + (i - start[s])};
}

// Scene s of a batch as a single-call argument set with B = 1.
__device__ __forceinline__ OpArgs scene_view(const BatchArgs& b, int s, int feat_bytes) {
    const msda_scene& sc = b.scenes[s];
    OpArgs a = {};
    a.feat = sc.feat;
    a.shapes = sc.spatial_shapes;
    a.starts = sc.level_start_index;
    a.loc = sc.sampling_loc;
    // under a weight flag: the FP32 weights (backward), or the scene's
    // logits / BF16 weights with its anchors' softmax statistics (forward)
    a.w = b.w32 ? b.w32 + (size_t)b.t.sample_start[s] * (size_t)b.G : sc.weights;
    a.w_bf16 = b.w32 ? 0 : b.w_bf16;
    a.wstats = (b.w32 || !b.wstats) ? nullptr : b.wstats + (size_t)b.t.anchor_start[s] * (size_t)b.G;
    a.level_scale = b.level_scale;
    a.grad_out = sc.grad_out;
    a.out = sc.out;
    a.grad_loc = sc.grad_sampling_loc;
    a.grad_w = sc.grad_weights;
    a.rec_key = b.rec_key;
    a.rec_frac = b.rec_frac;
    a.cell_start = b.rec_key ? b.t.cell_start + b.t.region_start[s] : nullptr;
    a.cells_per_item = 0;
    a.cell_offset = 0;
    a.no_cell = b.total_cells;
    a.sample_offset = b.rec_key ? b.t.sample_start[s] : 0u;
    a.rec_bucket_ap = b.rec_key && b.rec_bucketed ? (u32)sc.num_anchors * (u32)b.P : 0u;
    a.B = 1;
    a.N = sc.num_cams;
    a.L = b.L;
    a.A = sc.num_anchors;
    a.P = b.P;
    a.C = b.C;
    a.G = b.G;
    a.R = sc.rows;
    a.batch_bytes = (u32)(sc.rows * (int64_t)b.C * feat_bytes);
    a.lps_shift = b.lps_shift;
    return a;
}

// Quotient of n < 2^30 by the divisor whose magic is (m, shift): exact
// (Granlund-Montgomery with a round-up multiplier, see divmagic()).
__device__ __forceinline__ u32 fast_div(u32 n, u64 m, int shift) {
    return (u32)(((u64)n * m) >> shift);
}

}  // namespace msda
