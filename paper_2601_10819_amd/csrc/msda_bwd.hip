// Backward gathers of multi-scale deformable aggregation: gradients of
// <grad_out, out> with respect to the sampling locations and the weights,
// and the grad_feat records.
//
// msda_bwd_kernel (one workgroup per (batch item, anchor)) and
// msda_bwd_view_kernel (view order) re-gather the 4 corner rows of each
// sample (msda_grads.h) and write grad_weights and grad_sampling_loc. For
// grad_feat they either emit one record per sample -- the bilinear cell the
// sample falls in (its top-left neighbour, (y0+1, x0+1) in an (H+1) x (W+1)
// grid per region) and its fractions (lx, ly) -- for the sorted, tiled
// reduction (msda_sort.hip, msda_tiles.hip; deterministic, no float atomics),
// or add w * cw * grad_out to an FP32 accumulator with float atomics.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "msda_grads.h"

namespace msda {

// The backward gather of one anchor (index ba = b*A + a of `a`) by the whole
// workgroup in anchor order: pair by pair to the waves in turn, camera by
// camera, so that all workgroups go through the cameras together and the L2s
// hold the ones they are at (a run of pairs per wave, keypoint by keypoint: 64
// cameras of 256 x 448, 900 anchors FP32 1342 us, BF16 667, now 1030 and 476; 16
// cameras 272 and 134, now 216 and 103; rig of 6 of 256 x 704 105 and 50, now 84
// and 44).
template <class FT, int CPL, bool PACKED>
__device__ __forceinline__ void bwd_anchor(const OpArgs& a, const int ba, unsigned char* smem) {
    const int wave = wave_index(), nwaves = blockDim.x >> 6, npairs = a.P * a.N;
    const int b = ba / a.A;
    grads_of<FT, CPL, PACKED>(a, grad_anchor<FT>(a, b, ba - b * a.A),
                              AnchorOrder{a.P, nwaves, wave, div_magic(a.P, npairs)}, 0,
                              (npairs - wave + nwaves - 1) / nwaves, lanes_of<FT, CPL>(a),
                              smem + (size_t)wave * grads_lds_bytes(a.G));
}

template <class FT, int CPL, bool PACKED>
__global__ void __launch_bounds__(512) msda_bwd_kernel(OpArgs a, int ba0) {
    extern __shared__ __align__(16) unsigned char smem[];
    bwd_anchor<FT, CPL, PACKED>(a, ba0 + (int)blockIdx.x, smem);
}

// View order: unit (b*rows + j)*A + a is anchor a over row j of `rows` rows of
// cameras of batch item b (bwd_rows), cut camera-major into one range per XCD.
// Every output is per sample or per pair, so the rows need no combining.
template <class FT, int CPL, bool PACKED>
__global__ void __launch_bounds__(512) msda_bwd_view_kernel(OpArgs a, SlotCuts cuts,
                                                            int rows) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int wave = wave_index(), nwaves = blockDim.x >> 6;
    const u64 u = slot_unit(cuts, blockIdx.x, wave, nwaves);
    if (u == kNoUnit) return;
    const RowUnit t = row_unit(u, a.A);
    const int b = (int)(t.row / (u32)rows);
    const CamRange n = row_cams(a.N, (int)(t.row % (u32)rows), rows);
    const int np = (n.hi - n.lo) * a.P;
    grads_of<FT, CPL, PACKED>(a, grad_anchor<FT>(a, b, t.a),
                      ViewOrder{a.P, n.lo, div_magic(a.P, np)}, 0, np, lanes_of<FT, CPL>(a),
                      smem + (size_t)wave * grads_lds_bytes(a.G));
}

// Batched backward gather: persistent workgroups stride over the anchors of
// all scenes; records go to the batch's sample space, per (scene, region)
// bucket with local cells or at the sample index with batch-global cells.
template <class FT, int CPL, bool PACKED>
__global__ void __launch_bounds__(512) msda_bwd_batched_kernel(BatchArgs b) {
    extern __shared__ __align__(16) unsigned char smem[];
    for (u32 item = blockIdx.x; item < b.total_anchors; item += gridDim.x) {
        const int s = scene_of(b.t.anchor_start, b.S, item);
        bwd_anchor<FT, CPL, PACKED>(scene_view(b, s, FT::kBytes),
                                    (int)(item - b.t.anchor_start[s]), smem);
    }
}

// Batched backward gather in view order: each scene's units cut into one range
// per XCD, an XCD's ranges one after the other.
template <class FT, int CPL, bool PACKED>
__global__ void __launch_bounds__(512) msda_bwd_batched_view_kernel(BatchArgs b) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int wave = wave_index(), nwaves = blockDim.x >> 6;
    const SceneUnit su = scene_unit(b, blockIdx.x, wave, nwaves);
    if (su.s < 0) return;
    const OpArgs a = scene_view(b, su.s, FT::kBytes);
    const RowUnit t = row_unit(su.u, a.A);
    const CamRange n = row_cams(a.N, (int)t.row, bwd_rows(a.N, a.P));
    const int np = (n.hi - n.lo) * a.P;
    grads_of<FT, CPL, PACKED>(a, grad_anchor<FT>(a, 0, t.a),
                      ViewOrder{a.P, n.lo, div_magic(a.P, np)}, 0, np, lanes_of<FT, CPL>(a),
                      smem + (size_t)wave * grads_lds_bytes(a.G));
}

size_t gather_lds_bytes(int waves, int C, int G) {
    // the backward's staging is the larger, but for the forward's wave sums
    const size_t red = (size_t)waves * C * sizeof(float), g = (size_t)waves * grads_lds_bytes(G);
    return g > red ? g : red;
}

// ---------------------------------------------------------------- launchers

template <class FT, int CPL>
static hipError_t bwd_launch(const OpArgs& a, int waves, hipStream_t s) {
    const auto kernel = a.G <= kPackedGroups ? msda_bwd_kernel<FT, CPL, true>
                                              : msda_bwd_kernel<FT, CPL, false>;
    return anchor_parts(a, waves, [&](int ba0, unsigned anchors) {
        mark_begin("msda_bwd_kernel", s);
        hipLaunchKernelGGL(kernel, dim3(anchors), dim3(64 * waves),
                           (size_t)waves * grads_lds_bytes(a.G), s, a, ba0);
        mark_end(s);
    });
}

hipError_t launch_backward(const OpArgs& a, int dtype, int cpl, int waves, hipStream_t s) {
    switch (dtype * 100 + cpl) {
        case kF32 * 100 + 1: return bwd_launch<TF32, 1>(a, waves, s);
        case kF32 * 100 + 2: return bwd_launch<TF32, 2>(a, waves, s);
        case kF32 * 100 + 4: return bwd_launch<TF32, 4>(a, waves, s);
        case kBF16 * 100 + 2: return bwd_launch<TBF16, 2>(a, waves, s);
        case kF16 * 100 + 2: return bwd_launch<TF16, 2>(a, waves, s);
        case kBF16 * 100 + 4: return bwd_launch<TBF16, 4>(a, waves, s);
        case kF16 * 100 + 4: return bwd_launch<TF16, 4>(a, waves, s);
        case kBF16 * 100 + 8: return bwd_launch<TBF16, 8>(a, waves, s);
        case kF16 * 100 + 8: return bwd_launch<TF16, 8>(a, waves, s);
        default: return hipErrorInvalidValue;
    }
}

template <class FT, int CPL>
static hipError_t bwd_view_launch(const OpArgs& a, int waves, hipStream_t s) {
    const auto kernel = a.G <= kPackedGroups ? msda_bwd_view_kernel<FT, CPL, true>
                                              : msda_bwd_view_kernel<FT, CPL, false>;
    const int rows = bwd_rows(a.N, a.P);
    const SlotCuts cuts = UnitGroup{a.B, a.N, a.A, rows, 0, rows}.cuts();
    for (u64 at = 0; at < cuts.most(); at += kMaxSlotUnits) {
        mark_begin("msda_bwd_view_kernel", s);
        hipLaunchKernelGGL(kernel, dim3(slot_blocks(cuts.most() - at, waves)), dim3(64 * waves),
                           (size_t)waves * grads_lds_bytes(a.G), s, a, cuts.part(at), rows);
        mark_end(s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_backward_view(const OpArgs& a, int dtype, int cpl, int waves, hipStream_t s) {
    switch (dtype * 100 + cpl) {
        case kF32 * 100 + 1: return bwd_view_launch<TF32, 1>(a, waves, s);
        case kF32 * 100 + 2: return bwd_view_launch<TF32, 2>(a, waves, s);
        case kF32 * 100 + 4: return bwd_view_launch<TF32, 4>(a, waves, s);
        case kBF16 * 100 + 2: return bwd_view_launch<TBF16, 2>(a, waves, s);
        case kF16 * 100 + 2: return bwd_view_launch<TF16, 2>(a, waves, s);
        case kBF16 * 100 + 4: return bwd_view_launch<TBF16, 4>(a, waves, s);
        case kF16 * 100 + 4: return bwd_view_launch<TF16, 4>(a, waves, s);
        case kBF16 * 100 + 8: return bwd_view_launch<TBF16, 8>(a, waves, s);
        case kF16 * 100 + 8: return bwd_view_launch<TF16, 8>(a, waves, s);
        default: return hipErrorInvalidValue;
    }
}

template <class FT, int CPL>
static hipError_t bwd_batched_launch(const BatchArgs& b, int waves, int blocks, hipStream_t s) {
    const auto kernel = b.G <= kPackedGroups ? msda_bwd_batched_kernel<FT, CPL, true>
                                              : msda_bwd_batched_kernel<FT, CPL, false>;
    mark_begin("msda_bwd_batched_kernel", s);
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64 * waves),
                       (size_t)waves * grads_lds_bytes(b.G), s, b);
    mark_end(s);
    return hipGetLastError();
}

template <class FT, int CPL>
static hipError_t bwd_batched_view_launch(BatchArgs b, int waves, hipStream_t s) {
    const auto kernel = b.G <= kPackedGroups ? msda_bwd_batched_view_kernel<FT, CPL, true>
                                              : msda_bwd_batched_view_kernel<FT, CPL, false>;
    for (b.slot_begin = 0; b.slot_begin < b.slot_units; b.slot_begin += kMaxSlotUnits) {
        mark_begin("msda_bwd_batched_view_kernel", s);
        hipLaunchKernelGGL(kernel, dim3(slot_blocks(b.slot_units - b.slot_begin, waves)),
                           dim3(64 * waves), (size_t)waves * grads_lds_bytes(b.G), s, b);
        mark_end(s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_backward_batched_view(const BatchArgs& b, int dtype, int cpl, int waves,
                                        hipStream_t s) {
    switch (dtype * 100 + cpl) {
        case kF32 * 100 + 1: return bwd_batched_view_launch<TF32, 1>(b, waves, s);
        case kF32 * 100 + 2: return bwd_batched_view_launch<TF32, 2>(b, waves, s);
        case kF32 * 100 + 4: return bwd_batched_view_launch<TF32, 4>(b, waves, s);
        case kBF16 * 100 + 2: return bwd_batched_view_launch<TBF16, 2>(b, waves, s);
        case kF16 * 100 + 2: return bwd_batched_view_launch<TF16, 2>(b, waves, s);
        case kBF16 * 100 + 4: return bwd_batched_view_launch<TBF16, 4>(b, waves, s);
        case kF16 * 100 + 4: return bwd_batched_view_launch<TF16, 4>(b, waves, s);
        case kBF16 * 100 + 8: return bwd_batched_view_launch<TBF16, 8>(b, waves, s);
        case kF16 * 100 + 8: return bwd_batched_view_launch<TF16, 8>(b, waves, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_backward_batched(const BatchArgs& b, int dtype, int cpl, int waves, int blocks,
                                   hipStream_t s) {
    switch (dtype * 100 + cpl) {
        case kF32 * 100 + 1: return bwd_batched_launch<TF32, 1>(b, waves, blocks, s);
        case kF32 * 100 + 2: return bwd_batched_launch<TF32, 2>(b, waves, blocks, s);
        case kF32 * 100 + 4: return bwd_batched_launch<TF32, 4>(b, waves, blocks, s);
        case kBF16 * 100 + 2: return bwd_batched_launch<TBF16, 2>(b, waves, blocks, s);
        case kF16 * 100 + 2: return bwd_batched_launch<TF16, 2>(b, waves, blocks, s);
        case kBF16 * 100 + 4: return bwd_batched_launch<TBF16, 4>(b, waves, blocks, s);
        case kF16 * 100 + 4: return bwd_batched_launch<TF16, 4>(b, waves, blocks, s);
        case kBF16 * 100 + 8: return bwd_batched_launch<TBF16, 8>(b, waves, blocks, s);
        case kF16 * 100 + 8: return bwd_batched_launch<TF16, 8>(b, waves, blocks, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace msda
