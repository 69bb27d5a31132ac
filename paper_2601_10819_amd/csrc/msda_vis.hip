// Keypoint projection and the visible-view form of MSDA (paper Sec. 3.1,
// Sec. 3.2).
//
// project_keypoints_kernel: one thread per (batch item, anchor, camera)
// places the anchor's keypoints in the world -- box centre + yaw rotation
// of the box-frame offset scaled by (w, l, h) + velocity * dt (the motion
// compensation) -- projects them with the camera's 3x4 matrix, writes the
// normalised sampling locations (a point at or behind the camera gets a
// location outside every level) and whether any keypoint lands in the
// image: the anchor's visibility in that camera.
//
// Visible-view MSDA: only the (batch item, camera, anchor) items flagged
// visible are computed. The flags are compacted in view-major order (a scan
// of the flags gives each visible item its place), so consecutive items
// share a camera; the persistent gathers cut the item list into one range
// per XCD (as the view order does) and each wave takes one item at a time:
// the anchor's keypoints in that camera, all levels. The forward writes one
// partial row per item and fwd_visible_reduce adds an anchor's items in
// camera order; the backward writes grad_w / grad_loc of the visible pairs
// and one compacted grad_feat record per sample, which the sort and the
// tile reduction of the dense backward then consume.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "msda_grads.h"
#include "msda_rows.h"

namespace msda {

constexpr float kDepthEps = 1e-5f;
constexpr float kBehind = -2.0f;   // a location outside every level

__global__ void __launch_bounds__(256) project_keypoints_kernel(ProjArgs p) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t total = (size_t)p.B * p.A * p.N;
    if (t >= total) return;
    const int n = (int)(t % (size_t)p.N);
    const size_t ba = t / (size_t)p.N;                 // b * A + a
    const int b = (int)(ba / (size_t)p.A);
    const float* an = p.anchors + ba * 10;
    const float x = an[0], y = an[1], z = an[2], w = an[3], l = an[4], h = an[5];
    const float yaw = an[6];
    const float mx = p.dt * an[7], my = p.dt * an[8], mz = p.dt * an[9];
    float sy, cy;
    sincosf(yaw, &sy, &cy);
    const float* M = p.projection + ((size_t)b * p.N + n) * 12;
    const float W = (float)p.image_hw[2 * n + 1], H = (float)p.image_hw[2 * n];
    bool seen = false;
    for (int k = 0; k < p.P; ++k) {
        const float* kp = p.keypoints + (ba * p.P + k) * 3;
        const float ox = kp[0] * w, oy = kp[1] * l, oz = kp[2] * h;
        const float X = x + (cy * ox - sy * oy) + mx;
        const float Y = y + (sy * ox + cy * oy) + my;
        const float Z = z + oz + mz;
        const float u = M[0] * X + M[1] * Y + M[2] * Z + M[3];
        const float v = M[4] * X + M[5] * Y + M[6] * Z + M[7];
        const float d = M[8] * X + M[9] * Y + M[10] * Z + M[11];
        float lu = kBehind, lv = kBehind;
        if (d > kDepthEps) {
            const float px = u / d, py = v / d;
            lu = px / W;
            lv = py / H;
            seen |= px >= 0.f && px < W && py >= 0.f && py < H;
        }
        float* dst = p.loc + ((ba * p.P + k) * p.N + n) * 2;
        dst[0] = lu;
        dst[1] = lv;
    }
    p.visible[t] = seen ? 1 : 0;
}

hipError_t launch_project_keypoints(const ProjArgs& p, hipStream_t s) {
    const size_t total = (size_t)p.B * p.A * p.N;
    if (total == 0) return hipSuccess;
    mark_begin("project_keypoints", s);
    hipLaunchKernelGGL(project_keypoints_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256),
                       0, s, p);
    mark_end(s);
    return hipGetLastError();
}

// The compaction: blocks of kVisTile view-major items v = (b*N + n)*A + a,
// kVisItems consecutive ones per thread. visible_count_kernel writes the
// blocks' totals, and each block of visible_place_kernel adds those before it
// (as many words as there are blocks, out of the L2) instead of a launch that
// scans them; up to kVisTile - 1 items are one block and one launch. Bound by
// launches: 4 cameras of 545 anchors 14 -> 7.5 us, 64 of 900 23 -> 10, with
// the flags, a scan of three launches and the items before.
constexpr int kVisItems = 8;
constexpr int kVisTile = 256 * kVisItems;

// Bit k: item v0 + k is visible (v0 + k < V).
__device__ __forceinline__ u32 visible_bits(const uint8_t* __restrict__ visible, size_t v0,
                                            size_t V, int N, int A) {
    u32 seen[kVisItems];
#pragma unroll
    for (int k = 0; k < kVisItems; ++k) {
        const u32 v = (u32)(v0 + k < V ? v0 + k : V - 1);       // (items are 32-bit)
        const u32 bn = v / (u32)A, a = v - bn * (u32)A;
        const u32 b = bn / (u32)N, n = bn - b * (u32)N;
        seen[k] = visible[((size_t)b * (u32)A + a) * (u32)N + n];
    }
    u32 bits = 0;
#pragma unroll
    for (int k = 0; k < kVisItems; ++k)
        if (v0 + k < V && seen[k]) bits |= 1u << k;
    return bits;
}

__global__ void __launch_bounds__(256) visible_count_kernel(const uint8_t* __restrict__ visible,
                                                            size_t V, int N, int A,
                                                            u32* __restrict__ partial) {
    __shared__ u32 lds4[4];
    const size_t v0 = (size_t)blockIdx.x * kVisTile + threadIdx.x * (u32)kVisItems;
    u32 total;
    block_inclusive_scan(__popc(visible_bits(visible, v0, V, N, A)), lds4, &total);
    if (threadIdx.x == 0) partial[blockIdx.x] = total;
}

// place[0..V], items and rec_count (see launch_visible_items) of one block.
__global__ void __launch_bounds__(256) visible_place_kernel(const uint8_t* __restrict__ visible,
                                                            const u32* __restrict__ partial,
                                                            size_t V, int N, int A, u32 per_item,
                                                            u32* __restrict__ place,
                                                            u32* __restrict__ items,
                                                            u32* __restrict__ rec_count) {
    __shared__ u32 lds4[4];
    u32 mine = 0, before;
    for (u32 i = threadIdx.x; i < blockIdx.x; i += blockDim.x) mine += partial[i];
    block_inclusive_scan(mine, lds4, &before);
    const size_t v0 = (size_t)blockIdx.x * kVisTile + threadIdx.x * (u32)kVisItems;
    const u32 bits = visible_bits(visible, v0, V, N, A);
    u32 total;
    u32 at = before + block_inclusive_scan(__popc(bits), lds4, &total) - __popc(bits);
#pragma unroll
    for (int k = 0; k < kVisItems; ++k) {
        if (v0 + k > V) break;
        place[v0 + k] = at;
        if (v0 + k == V && rec_count) rec_count[0] = at * per_item;
        if (bits >> k & 1) items[at++] = (u32)(v0 + k);
    }
}

// Visibility-weighted fusion (Sec. 3.2, Eq. 2). One wave per (batch item,
// anchor); V = the sum of the scores of the anchor's visible cameras, added
// lane-strided then by a fixed butterfly (the same order in every pass).
__device__ __forceinline__ float wave_score_sum(const uint8_t* visible, const float* score,
                                                size_t o, int N, int lane) {
    float V = 0.f;
    for (int n = lane; n < N; n += 64)
        if (visible[o + n]) V += score[o + n];
    return group_sum(V, 64);
}

// vt[b][a][n] = score / V for visible cameras; 0 for the others, and for
// every camera when V <= 0.
__global__ void __launch_bounds__(256) view_scale_kernel(const uint8_t* __restrict__ visible,
                                                         const float* __restrict__ score,
                                                         int BA, int N, float* __restrict__ vt) {
    const int ba = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (ba >= BA) return;                     // whole waves
    const size_t o = (size_t)ba * N;
    const float V = wave_score_sum(visible, score, o, N, lane);
    for (int n = lane; n < N; n += 64)
        vt[o + n] = visible[o + n] && V > 0.f ? score[o + n] / V : 0.f;
}

// grad_score[b][a][n] = (<grad_out, g_n> - <grad_out, f>) / V for visible
// cameras (0 otherwise, and when V <= 0): g_n's product with grad_out comes
// from the backward gather (item_dot), f is the fused forward output.
__global__ void __launch_bounds__(256) grad_score_kernel(const float* __restrict__ grad_out,
                                                         const float* __restrict__ out,
                                                         const uint8_t* __restrict__ visible,
                                                         const float* __restrict__ score,
                                                         const u32* __restrict__ place,
                                                         const float* __restrict__ item_dot,
                                                         int B, int A, int N, int C,
                                                         float* __restrict__ grad_score) {
    const int ba = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (ba >= B * A) return;                  // whole waves
    const int b = ba / A, an = ba - b * A;
    const size_t o = (size_t)ba * N;
    const float V = wave_score_sum(visible, score, o, N, lane);
    float fdot = 0.f;
    for (int c = lane; c < C; c += 64)
        fdot = fmaf(grad_out[(size_t)ba * C + c], out[(size_t)ba * C + c], fdot);
    fdot = group_sum(fdot, 64);
    for (int n = lane; n < N; n += 64) {
        float gs = 0.f;
        if (visible[o + n] && V > 0.f) {
            const u32 i = place[((size_t)b * N + n) * A + an];
            gs = (item_dot[i] - fdot) / V;
        }
        grad_score[o + n] = gs;
    }
}

// The persistent walk over the visible items: workgroup w serves range
// w % kSlots of the item list; its waves take consecutive items, then move
// on by the slot's wave count. Calls f(item index, b, a, n) per item.
template <class F>
__device__ __forceinline__ void for_each_visible_item(const OpArgs& a, const u32* items,
                                                      const u32* count, F&& f) {
    const u32 nnz = uniform((int)*count);
    const int x = (int)(blockIdx.x % kSlots);
    const int wave = wave_index(), nwaves = blockDim.x >> 6;
    const u32 lo = (u32)(((u64)nnz * x) / kSlots), hi = (u32)(((u64)nnz * (x + 1)) / kSlots);
    const u32 per_slot = (gridDim.x / kSlots + (x < (int)(gridDim.x % kSlots) ? 1u : 0u));
    const u32 stride = per_slot * (u32)nwaves;
    for (u32 r = (blockIdx.x / kSlots) * (u32)nwaves + (u32)wave; lo + r < hi; r += stride) {
        const u32 i = lo + r;
        const u32 v = uniform((int)items[i]);
        const int an = (int)(v % (u32)a.A);
        const u32 bn = v / (u32)a.A;
        f(i, (int)(bn / (u32)a.N), an, (int)(bn % (u32)a.N));
    }
}

template <class FT, int CPL, bool PACKED>
__global__ void __launch_bounds__(512) msda_fwd_visible_kernel(OpArgs a, const u32* items,
                                                               const u32* count, int chunk,
                                                               float* part) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Lanes q = lanes_of<FT, CPL>(a);
    unsigned char* lds = smem + (size_t)wave_index() * row_lds_bytes(chunk, a.G);
    const int NS = a.P * a.L;
    for_each_visible_item(a, items, count, [&](u32 i, int b, int an, int n) {
        const rsrc_t feat = make_rsrc(static_cast<const char*>(a.feat) + (size_t)b * a.batch_bytes,
                                      a.batch_bytes);
        float acc[CPL];
        row_sum<FT, CPL, PACKED>(a, (size_t)b * a.A + an, feat, n * NS, (n + 1) * NS, q, chunk,
                                 lds, acc);
        if (q.sub == 0) {
            float* dst = part + (size_t)i * a.C + q.c0;
#pragma unroll
            for (int c = 0; c < CPL; ++c) dst[c] = acc[c];
        }
    });
}

// out[b, a, :] = sum over the anchor's visible cameras, in camera order, of
// the items' partial rows, each times vt (the fused form's per-view weight)
// when vt is given; zero when no camera sees the anchor. One wave per
// anchor, 4 channels per lane per pass: a ballot of the visibility flags
// of 64 cameras, then the items' rows 4 at a time (loads in flight
// together, added in camera order).
__global__ void __launch_bounds__(256) fwd_visible_reduce(const float* __restrict__ part,
                                                          const uint8_t* __restrict__ visible,
                                                          const u32* __restrict__ place,
                                                          const float* __restrict__ vt, int B,
                                                          int N, int A, int C,
                                                          float* __restrict__ out) {
    const int ba = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (ba >= B * A) return;                  // whole waves
    const int b = ba / A, an = ba - b * A;
    const size_t o = (size_t)ba * N;
    for (int c0 = 0; c0 < C; c0 += 256) {
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        for (int n0 = 0; n0 < N; n0 += 64) {
            const int n = n0 + lane;
            const bool f = n < N && visible[o + n];
            const u32 pl = f ? place[((size_t)b * N + n) * A + an] : 0u;
            const float sc = f && vt ? vt[o + n] : 1.f;
            uint64_t mask = __ballot(f);
            while (mask) {
                int k[4];
                int m = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    k[q] = mask ? __builtin_ctzll(mask) : 0;
                    if (mask) { mask &= mask - 1; ++m; }
                }
                float g[4][4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const u32 i = (u32)__shfl((int)pl, k[q], 64);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int c = c0 + lane + 64 * j;
                        g[q][j] = q < m && c < C ? part[(size_t)i * C + c] : 0.f;
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    if (q >= m) break;
                    const float w = __shfl(sc, k[q], 64);
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[j] = vt ? fmaf(w, g[q][j], acc[j]) : acc[j] + g[q][j];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = c0 + lane + 64 * j;
            if (c < C) out[(size_t)ba * C + c] = acc[j];
        }
    }
}

template <class FT, int CPL, bool PACKED>
__global__ void __launch_bounds__(512) msda_bwd_visible_kernel(OpArgs a, const u32* items,
                                                               const u32* place,
                                                               const u32* count,
                                                               u32* rec_val, const float* vt,
                                                               float* item_dot) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Lanes q = lanes_of<FT, CPL>(a);
    unsigned char* lds = smem + (size_t)wave_index() * grads_lds_bytes(a.G);
    const u32 mP = div_magic(a.P, a.P);
    for_each_visible_item(a, items, count, [&](u32 i, int b, int an, int n) {
        GradAnchor x = grad_anchor<FT>(a, b, an);
        if (a.rec_bucket_ap) {
            // records per (b, n, l) bucket (launch_bucket_sort's visible-view
            // layout): the cnt visible anchors of (b, n) from item s0 on,
            // level-major; stage_grads adds (n*L + l)*ap + p, so the base
            // drops n*L*ap (modulo 2^32)
            const u32 bn = (u32)(b * a.N + n), P = (u32)a.P, L = (u32)a.L;
            const u32 s0 = place[(size_t)bn * a.A];
            x.rec.ap = (place[(size_t)(bn + 1) * a.A] - s0) * P;
            x.rec.bucket_base = s0 * P * L + (i - s0) * P - (u32)n * L * x.rec.ap;
        } else {
            x.rec.val = rec_val;
            x.rec.cbase = i * (u32)(a.P * a.L);
        }
        const float scale = vt ? vt[((size_t)b * a.A + an) * a.N + n] : 1.f;
        float dot = 0.f;
        grads_of<FT, CPL, PACKED>(a, x, ViewOrder{a.P, n, mP}, 0, a.P, q, lds, scale,
                          item_dot ? &dot : nullptr);
        if (item_dot) {
            dot = group_sum(dot, 64);
            if (q.lane == 0) item_dot[i] = dot;
        }
    });
}

// Persistent grids: 16 workgroups of `waves` waves per CU's worth of slots,
// rounded to whole slots.
static unsigned visible_blocks(int waves) {
    const unsigned per_cu = 16u / (unsigned)waves > 0 ? 16u / (unsigned)waves : 1u;
    return 256u * per_cu / kSlots * kSlots;
}

template <class FT, int CPL>
static hipError_t fwd_visible_launch(const OpArgs& a, int waves, const u32* items,
                                     const u32* count, const u32* place, const uint8_t* visible,
                                     const float* vt, float* part, hipStream_t s) {
    const int chunk = fwd_chunk_samples(waves, a.G);
    const auto kernel = a.G <= kPackedGroups ? msda_fwd_visible_kernel<FT, CPL, true>
                                              : msda_fwd_visible_kernel<FT, CPL, false>;
    mark_begin("msda_fwd_visible_kernel", s);
    hipLaunchKernelGGL(kernel, dim3(visible_blocks(waves)),
                       dim3(64 * waves), (size_t)waves * row_lds_bytes(chunk, a.G), s, a, items,
                       count, chunk, part);
    mark_end(s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t anchors = (size_t)a.B * a.A;
    mark_begin("fwd_visible_reduce", s);
    hipLaunchKernelGGL(fwd_visible_reduce, dim3((unsigned)((anchors + 3) / 4)), dim3(256), 0, s,
                       part, visible, place, vt, a.B, a.N, a.A, a.C, a.out);
    mark_end(s);
    return hipGetLastError();
}

template <class FT, int CPL>
static hipError_t bwd_visible_launch(const OpArgs& a, int waves, const u32* items,
                                     const u32* place, const u32* count, u32* rec_val,
                                     const float* vt, float* item_dot, hipStream_t s) {
    const auto kernel = a.G <= kPackedGroups ? msda_bwd_visible_kernel<FT, CPL, true>
                                              : msda_bwd_visible_kernel<FT, CPL, false>;
    mark_begin("msda_bwd_visible_kernel", s);
    hipLaunchKernelGGL(kernel, dim3(visible_blocks(waves)),
                       dim3(64 * waves), (size_t)waves * grads_lds_bytes(a.G), s, a, items, place,
                       count, rec_val, vt, item_dot);
    mark_end(s);
    return hipGetLastError();
}

size_t visible_partial_words(size_t V) { return V / kVisTile + 1; }

hipError_t launch_visible_items(const uint8_t* visible, int B, int N, int A, u32 per_item,
                                u32* place, u32* items, u32* rec_count, u32* partial,
                                hipStream_t s) {
    const size_t V = (size_t)B * N * A;
    const unsigned blocks = (unsigned)(V / kVisTile + 1);      // items 0..V
    if (blocks > 1) {
        mark_begin("visible_count", s);
        hipLaunchKernelGGL(visible_count_kernel, dim3(blocks), dim3(256), 0, s, visible, V, N, A,
                           partial);
        mark_end(s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    mark_begin("visible_place", s);
    hipLaunchKernelGGL(visible_place_kernel, dim3(blocks), dim3(256), 0, s, visible, partial, V, N,
                       A, per_item, place, items, rec_count);
    mark_end(s);
    return hipGetLastError();
}

hipError_t launch_forward_visible(const OpArgs& a, int dtype, int cpl, int waves,
                                  const u32* items, const u32* count, const u32* place,
                                  const uint8_t* visible, const float* vt, float* part,
                                  hipStream_t s) {
    switch (dtype * 100 + cpl) {
#define MSDA_CASE(D, T, K) \
        case D * 100 + K: \
            return fwd_visible_launch<T, K>(a, waves, items, count, place, visible, vt, \
                                            part, s);
        MSDA_CASE(kF32, TF32, 1) MSDA_CASE(kF32, TF32, 2) MSDA_CASE(kF32, TF32, 4)
        MSDA_CASE(kBF16, TBF16, 2) MSDA_CASE(kBF16, TBF16, 4) MSDA_CASE(kBF16, TBF16, 8)
        MSDA_CASE(kF16, TF16, 2) MSDA_CASE(kF16, TF16, 4) MSDA_CASE(kF16, TF16, 8)
        MSDA_CASE(kFP8, TFP8, 4) MSDA_CASE(kFP8, TFP8, 8) MSDA_CASE(kFP8, TFP8, 16)
#undef MSDA_CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_backward_visible(const OpArgs& a, int dtype, int cpl, int waves,
                                   const u32* items, const u32* place, const u32* count,
                                   u32* rec_val, const float* vt, float* item_dot, hipStream_t s) {
    switch (dtype * 100 + cpl) {
#define MSDA_CASE(D, T, K) \
        case D * 100 + K: \
            return bwd_visible_launch<T, K>(a, waves, items, place, count, rec_val, vt, \
                                            item_dot, s);
        MSDA_CASE(kF32, TF32, 1) MSDA_CASE(kF32, TF32, 2) MSDA_CASE(kF32, TF32, 4)
        MSDA_CASE(kBF16, TBF16, 2) MSDA_CASE(kBF16, TBF16, 4) MSDA_CASE(kBF16, TBF16, 8)
        MSDA_CASE(kF16, TF16, 2) MSDA_CASE(kF16, TF16, 4) MSDA_CASE(kF16, TF16, 8)
#undef MSDA_CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_view_scale(const uint8_t* visible, const float* score, int BA, int N,
                             float* vt, hipStream_t s) {
    if (BA <= 0) return hipSuccess;
    mark_begin("view_scale", s);
    hipLaunchKernelGGL(view_scale_kernel, dim3((unsigned)((BA + 3) / 4)), dim3(256), 0, s,
                       visible, score, BA, N, vt);
    mark_end(s);
    return hipGetLastError();
}

hipError_t launch_grad_score(const float* grad_out, const float* out, const uint8_t* visible,
                             const float* score, const u32* place, const float* item_dot, int B,
                             int A, int N, int C, float* grad_score, hipStream_t s) {
    if (B * A <= 0) return hipSuccess;
    mark_begin("grad_score", s);
    hipLaunchKernelGGL(grad_score_kernel, dim3((unsigned)((B * A + 3) / 4)), dim3(256), 0, s,
                       grad_out, out, visible, score, place, item_dot, B, A, N, C, grad_score);
    mark_end(s);
    return hipGetLastError();
}

}  // namespace msda
