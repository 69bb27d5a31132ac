// Forward kernels of multi-scale deformable aggregation (paper Sec. 3.1 /
// Sec. 3.2): out[b,a,:] = sum over (keypoint, camera, level) of weight *
// bilinear sample.
//
// Anchor order (msda_fwd_kernel): one workgroup per (batch item, anchor);
// its waves split the anchor's samples and the waves' partial sums are added
// in a fixed order at the end.
//
// View order (msda_fwd_view_kernel): the rows -- a run of cameras, see
// fwd_rows -- of every anchor are cut, camera-major, into one contiguous
// range per XCD; each wave sums one anchor over one row and writes a partial
// row, and fwd_rows_reduce adds an anchor's rows in order. Both orders are
// deterministic.
//
// In both, a wave stages its samples one per lane, so the coordinate
// arithmetic is done once per sample rather than once per lane of a sample,
// then each group of C/CPL lanes takes a sample at a time and issues several
// samples' corner loads before using them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "msda_rows.h"

namespace msda {

// The forward of one anchor (index ba = b*A + a of `a`) by the whole
// workgroup in anchor order. Called by every thread of the block (it ends
// with block-wide barriers).
template <class FT, int CPL, bool PACKED>
__device__ __forceinline__ void fwd_anchor(const OpArgs& a, const int ba, int chunk,
                                           unsigned char* smem) {
    const int wave = wave_index(), nwaves = blockDim.x >> 6;
    const Lanes q = lanes_of<FT, CPL>(a);
    const int b = ba / a.A;
    const rsrc_t feat = make_rsrc(static_cast<const char*>(a.feat) + (size_t)b * a.batch_bytes,
                                  a.batch_bytes);
    // equal runs of samples, of whole chunks of 64 where there are several
    const int total = a.P * a.N * a.L;
    int per = (total + nwaves - 1) / nwaves;
    if (per > 64) per = (per + 63) & ~63;
    const int s_lo = (int)min((int64_t)total, (int64_t)wave * per);
    float acc[CPL];
    row_sum<FT, CPL, PACKED>(a, (size_t)ba, feat, s_lo, min(total, s_lo + per), q, chunk,
                     smem + (size_t)wave * row_lds_bytes(chunk, a.G), acc);

    float* out = a.out + (size_t)ba * a.C;
    if (nwaves == 1) {
        if (q.sub == 0) {
#pragma unroll
            for (int i = 0; i < CPL; ++i) out[q.c0 + i] = acc[i];
        }
        return;
    }
    float* red = reinterpret_cast<float*>(smem);
    __syncthreads();                       // every wave is done with its staging
    if (q.sub == 0) {
#pragma unroll
        for (int i = 0; i < CPL; ++i) red[wave * a.C + q.c0 + i] = acc[i];
    }
    __syncthreads();
    for (int c = threadIdx.x; c < a.C; c += blockDim.x) {
        float s = 0.f;
        for (int w = 0; w < nwaves; ++w) s += red[w * a.C + c];   // fixed order
        out[c] = s;
    }
    __syncthreads();                       // smem is free again
}

// LDS of an anchor-order workgroup: the waves' staging, then their sums.
static size_t anchor_lds_bytes(int waves, int chunk, int C, int G) {
    const size_t stage = (size_t)waves * row_lds_bytes(chunk, G);
    const size_t red = (size_t)waves * C * sizeof(float);
    return stage > red ? stage : red;
}

template <class FT, int CPL, bool PACKED>
__global__ void __launch_bounds__(512) msda_fwd_kernel(OpArgs a, int ba0, int chunk) {
    extern __shared__ __align__(16) unsigned char smem[];
    fwd_anchor<FT, CPL, PACKED>(a, ba0 + (int)blockIdx.x, chunk, smem);
}

// View order: rows [row0, row0 + nrows) of every batch item, of `rows` in
// all; unit (b*nrows + j)*A + a, the partial row of that index in part.
template <class FT, int CPL, bool PACKED>
__global__ void __launch_bounds__(512) msda_fwd_view_kernel(OpArgs a, SlotCuts cuts,
                                                            int rows, int row0, int nrows,
                                                            int chunk, float* part) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int wave = wave_index(), nwaves = blockDim.x >> 6;
    const u64 u = slot_unit(cuts, blockIdx.x, wave, nwaves);
    if (u == kNoUnit) return;
    const RowUnit t = row_unit(u, a.A);
    const int b = (int)(t.row / (u32)nrows);
    const CamRange n = row_cams(a.N, row0 + (int)(t.row % (u32)nrows), rows);
    const Lanes q = lanes_of<FT, CPL>(a);
    const rsrc_t feat = make_rsrc(
        static_cast<const char*>(a.feat) + (size_t)b * a.batch_bytes, a.batch_bytes);
    const int NS = a.P * a.L;
    float acc[CPL];
    row_sum<FT, CPL, PACKED>(a, (size_t)b * a.A + t.a, feat, n.lo * NS, n.hi * NS, q, chunk,
                     smem + (size_t)wave * row_lds_bytes(chunk, a.G), acc);
    if (q.sub == 0) {
        float* dst = part + u * (u32)a.C + q.c0;
#pragma unroll
        for (int i = 0; i < CPL; ++i) dst[i] = acc[i];
    }
}

// out[b][i] = the sum of batch item b's partial rows in row order (added to
// out with `more`: the rows after those already in it); four floats per
// thread (C % 4 == 0) or one.
template <int V>
__global__ void __launch_bounds__(256) fwd_rows_reduce(const float* part, float* out, int B,
                                                       int rows, size_t AC, bool more) {
    const size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * V;
    if (i >= (size_t)B * AC) return;
    const size_t b = i / AC;
    const float* p = part + b * rows * AC + (i - b * AC);
    float s[V];
#pragma unroll
    for (int v = 0; v < V; ++v) s[v] = more ? out[i + v] : 0.f;
#pragma unroll 8
    for (int x = 0; x < rows; ++x, p += AC) {
        if constexpr (V == 4) {
            const float4 t = *reinterpret_cast<const float4*>(p);
            s[0] += t.x; s[1] += t.y; s[2] += t.z; s[3] += t.w;
        } else {
            s[0] += p[0];
        }
    }
    if constexpr (V == 4) {
        *reinterpret_cast<float4*>(out + i) = make_float4(s[0], s[1], s[2], s[3]);
    } else {
        out[i] = s[0];
    }
}

// Batched forward: persistent workgroups stride over the anchors of all
// scenes.
template <class FT, int CPL, bool PACKED>
__global__ void __launch_bounds__(512) msda_fwd_batched_kernel(BatchArgs b, int chunk) {
    extern __shared__ __align__(16) unsigned char smem[];
    for (u32 item = blockIdx.x; item < b.total_anchors; item += gridDim.x) {
        const int s = scene_of(b.t.anchor_start, b.S, item);
        const OpArgs a = scene_view(b, s, FT::kBytes);
        fwd_anchor<FT, CPL, PACKED>(a, (int)(item - b.t.anchor_start[s]), chunk, smem);
    }
}

// Batched forward in view order: each scene's units cut into one range per XCD,
// as the single call's, and an XCD's ranges one after the other (one cut
// through all scenes left the XCDs whose scenes have larger maps behind: the
// 12-scene step 8.93 -> 8.62 ms, five scenes of 5 to 25 cameras FP32 135 ->
// 114 us, BF16 317 -> 263). Per anchor the arithmetic is the single call's view
// order with B = 1.
template <class FT, int CPL, bool PACKED>
__global__ void __launch_bounds__(512) msda_fwd_batched_view_kernel(BatchArgs b, int chunk,
                                                                    float* part) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int wave = wave_index(), nwaves = blockDim.x >> 6;
    const SceneUnit su = scene_unit(b, blockIdx.x, wave, nwaves);
    if (su.s < 0) return;
    const OpArgs a = scene_view(b, su.s, FT::kBytes);
    const RowUnit t = row_unit(su.u, a.A);
    const CamRange n = row_cams(a.N, (int)t.row, fwd_rows(a.N, a.P, a.L));
    const Lanes q = lanes_of<FT, CPL>(a);
    const rsrc_t feat = make_rsrc(a.feat, a.batch_bytes);
    const int NS = a.P * a.L;
    float acc[CPL];
    row_sum<FT, CPL, PACKED>(a, (size_t)t.a, feat, n.lo * NS, n.hi * NS, q, chunk,
                     smem + (size_t)wave * row_lds_bytes(chunk, a.G), acc);
    if (q.sub == 0) {
        float* dst = part + (b.t.row_start[su.s] + su.u) * (u32)b.C + q.c0;
#pragma unroll
        for (int i = 0; i < CPL; ++i) dst[i] = acc[i];
    }
}

// out of global anchor g = the sum of its partial rows in row order, written
// to its scene's output; V floats per thread.
template <int V>
__global__ void __launch_bounds__(256) fwd_batched_view_reduce(BatchArgs b, const float* part) {
    const size_t total = (size_t)b.total_anchors * b.C;
    const size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * V;
    if (i >= total) return;
    const u32 g = (u32)(i / (size_t)b.C);
    const int c = (int)(i - (size_t)g * b.C);
    const int sc = scene_of(b.t.anchor_start, b.S, g);
    const u32 a = g - b.t.anchor_start[sc];
    const size_t AC = (size_t)b.scenes[sc].num_anchors * b.C;
    const int rows = fwd_rows(b.scenes[sc].num_cams, b.P, b.L);
    const float* p = part + (b.t.row_start[sc] + a) * (u32)b.C + c;
    float s[V];
#pragma unroll
    for (int v = 0; v < V; ++v) s[v] = 0.f;
#pragma unroll 8
    for (int x = 0; x < rows; ++x, p += AC) {
        if constexpr (V == 4) {
            const float4 t = *reinterpret_cast<const float4*>(p);
            s[0] += t.x; s[1] += t.y; s[2] += t.z; s[3] += t.w;
        } else {
            s[0] += p[0];
        }
    }
    float* out = b.scenes[sc].out + (size_t)a * b.C + c;
    if constexpr (V == 4) {
        *reinterpret_cast<float4*>(out) = make_float4(s[0], s[1], s[2], s[3]);
    } else {
        out[0] = s[0];
    }
}

template <class FT, int CPL>
static hipError_t fwd_batched_view_launch(BatchArgs b, int waves, float* part, hipStream_t s) {
    const auto kernel = b.G <= kPackedGroups ? msda_fwd_batched_view_kernel<FT, CPL, true>
                                              : msda_fwd_batched_view_kernel<FT, CPL, false>;
    const int chunk = fwd_chunk_samples(waves, b.G);
    for (b.slot_begin = 0; b.slot_begin < b.slot_units; b.slot_begin += kMaxSlotUnits) {
        mark_begin("msda_fwd_batched_view_kernel", s);
        hipLaunchKernelGGL(kernel, dim3(slot_blocks(b.slot_units - b.slot_begin, waves)),
                           dim3(64 * waves), (size_t)waves * row_lds_bytes(chunk, b.G), s, b,
                           chunk, part);
        mark_end(s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const size_t total = (size_t)b.total_anchors * b.C;
    mark_begin("fwd_batched_view_reduce", s);
    if (b.C % 4 == 0) {
        hipLaunchKernelGGL(fwd_batched_view_reduce<4>, dim3((unsigned)((total / 4 + 255) / 256)),
                           dim3(256), 0, s, b, part);
    } else {
        hipLaunchKernelGGL(fwd_batched_view_reduce<1>, dim3((unsigned)((total + 255) / 256)),
                           dim3(256), 0, s, b, part);
    }
    mark_end(s);
    return hipGetLastError();
}

template <class FT, int CPL>
static hipError_t fwd_batched_launch(const BatchArgs& b, int waves, int blocks, hipStream_t s) {
    const int chunk = fwd_chunk_samples(waves, b.G);
    const auto kernel = b.G <= kPackedGroups ? msda_fwd_batched_kernel<FT, CPL, true>
                                              : msda_fwd_batched_kernel<FT, CPL, false>;
    mark_begin("msda_fwd_batched_kernel", s);
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * waves),
                       anchor_lds_bytes(waves, chunk, b.C, b.G), s, b, chunk);
    mark_end(s);
    return hipGetLastError();
}

template <class FT, int CPL>
static hipError_t fwd_launch(const OpArgs& a, int waves, hipStream_t s) {
    const auto kernel = a.G <= kPackedGroups ? msda_fwd_kernel<FT, CPL, true>
                                              : msda_fwd_kernel<FT, CPL, false>;
    const int chunk = fwd_chunk_samples(waves, a.G);
    return anchor_parts(a, waves, [&](int ba0, unsigned anchors) {
        mark_begin("msda_fwd_kernel", s);
        hipLaunchKernelGGL(kernel, dim3(anchors), dim3(64 * waves),
                           anchor_lds_bytes(waves, chunk, a.C, a.G), s, a, ba0, chunk);
        mark_end(s);
    });
}

template <class FT, int CPL>
static hipError_t fwd_view_launch(const OpArgs& a, int waves, int part_rows, float* part,
                                  hipStream_t s) {
    const auto kernel = a.G <= kPackedGroups ? msda_fwd_view_kernel<FT, CPL, true>
                                              : msda_fwd_view_kernel<FT, CPL, false>;
    const int rows = fwd_rows(a.N, a.P, a.L), chunk = fwd_chunk_samples(waves, a.G);
    const size_t AC = (size_t)a.A * a.C, total = AC * a.B;
    for (int row0 = 0; row0 < rows; row0 += part_rows) {
        const int nrows = part_rows < rows - row0 ? part_rows : rows - row0;
        const SlotCuts cuts = UnitGroup{a.B, a.N, a.A, rows, row0, nrows}.cuts();
        for (u64 at = 0; at < cuts.most(); at += kMaxSlotUnits) {
            mark_begin("msda_fwd_view_kernel", s);
            hipLaunchKernelGGL(kernel, dim3(slot_blocks(cuts.most() - at, waves)), dim3(64 * waves),
                               (size_t)waves * row_lds_bytes(chunk, a.G), s, a, cuts.part(at),
                               rows, row0, nrows, chunk, part);
            mark_end(s);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        mark_begin("fwd_rows_reduce", s);
        if (a.C % 4 == 0) {
            hipLaunchKernelGGL(fwd_rows_reduce<4>, dim3((unsigned)((total / 4 + 255) / 256)),
                               dim3(256), 0, s, part, a.out, a.B, nrows, AC, row0 > 0);
        } else {
            hipLaunchKernelGGL(fwd_rows_reduce<1>, dim3((unsigned)((total + 255) / 256)),
                               dim3(256), 0, s, part, a.out, a.B, nrows, AC, row0 > 0);
        }
        mark_end(s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Instantiations by (dtype, channels per lane).
#define MSDA_FOR_EACH_LAYOUT(F, ...)                                    \
    switch (dtype * 100 + cpl) {                                        \
        case kF32 * 100 + 1: return F<TF32, 1>(__VA_ARGS__);            \
        case kF32 * 100 + 2: return F<TF32, 2>(__VA_ARGS__);            \
        case kF32 * 100 + 4: return F<TF32, 4>(__VA_ARGS__);            \
        case kBF16 * 100 + 2: return F<TBF16, 2>(__VA_ARGS__);          \
        case kBF16 * 100 + 4: return F<TBF16, 4>(__VA_ARGS__);          \
        case kBF16 * 100 + 8: return F<TBF16, 8>(__VA_ARGS__);          \
        case kF16 * 100 + 2: return F<TF16, 2>(__VA_ARGS__);            \
        case kF16 * 100 + 4: return F<TF16, 4>(__VA_ARGS__);            \
        case kF16 * 100 + 8: return F<TF16, 8>(__VA_ARGS__);            \
        case kFP8 * 100 + 4: return F<TFP8, 4>(__VA_ARGS__);            \
        case kFP8 * 100 + 8: return F<TFP8, 8>(__VA_ARGS__);            \
        case kFP8 * 100 + 16: return F<TFP8, 16>(__VA_ARGS__);          \
        default: return hipErrorInvalidValue;                           \
    }

hipError_t launch_forward_batched(const BatchArgs& b, int dtype, int cpl, int waves, int blocks,
                                  hipStream_t s) {
    MSDA_FOR_EACH_LAYOUT(fwd_batched_launch, b, waves, blocks, s)
}

hipError_t launch_forward_batched_view(const BatchArgs& b, int dtype, int cpl, int waves,
                                       float* part, hipStream_t s) {
    MSDA_FOR_EACH_LAYOUT(fwd_batched_view_launch, b, waves, part, s)
}

hipError_t launch_forward(const OpArgs& a, int dtype, int cpl, int waves, hipStream_t s) {
    MSDA_FOR_EACH_LAYOUT(fwd_launch, a, waves, s)
}

hipError_t launch_forward_view(const OpArgs& a, int dtype, int cpl, int waves, int part_rows,
                               float* part, hipStream_t s) {
    MSDA_FOR_EACH_LAYOUT(fwd_view_launch, a, waves, part_rows, part, s)
}

}  // namespace msda
