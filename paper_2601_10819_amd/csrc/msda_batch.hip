// Tables of the batched form, built on the device from the scene table so
// that a batched call needs no host-to-device copy (and can be captured in
// a HIP graph): per scene the first anchor, sample (record) and region; per
// region its first bilinear cell; and the processing slots of the tiled
// grad_feat reduction -- sparse light levels last, of the rest wide scenes
// (BatchArgs::wide) first, then heavy (coarse) levels, then coarsest level
// first, then scene, then camera -- with the first tile of each slot.
//
// A scene's heavy regions are the first BatchArgs::heavy of its slots (coarsest
// level first, cameras in order), as the host counts them for the single call.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "msda_common.h"

namespace msda {

__global__ void __launch_bounds__(256) batch_tables_kernel(BatchArgs b, int backward) {
    __shared__ u32 s_anchors[kMaxBatchScenes];
    __shared__ u32 s_cams[kMaxBatchScenes];
    __shared__ u32 rstart[kMaxBatchScenes + 1];
    __shared__ uint16_t sh_h[kMaxBatchRegions];
    __shared__ uint16_t sh_w[kMaxBatchRegions];
    __shared__ u32 grp[2 * 8 * kMaxBatchScenes];    // first slot of (light, level, scene)
    __shared__ __align__(8) u32 tiles[kMaxBatchRegions];   // tiles of each slot, then their scan
    __shared__ u32 lds4[4];
    static_assert(2 * kSlots * kMaxBatchScenes <= kMaxBatchRegions, "slot_first is in tiles");
    u64* const slot_first = reinterpret_cast<u64*>(tiles); // first unit of (XCD slot, scene)
    const int S = b.S, L = b.L, tid = threadIdx.x;

    for (int s = tid; s < S; s += blockDim.x) {
        s_anchors[s] = (u32)b.scenes[s].num_anchors;
        s_cams[s] = (u32)b.scenes[s].num_cams;
    }
    __syncthreads();
    if (tid == 0) {
        u32 a = 0, smp = 0, reg = 0;
        u64 rows = 0;
        for (int s = 0; s < S; ++s) {
            b.t.anchor_start[s] = a;
            b.t.sample_start[s] = smp;
            b.t.region_start[s] = reg;
            rstart[s] = reg;
            b.t.row_start[s] = rows;
            const int N = (int)s_cams[s];
            rows += (u64)(backward ? bwd_rows(N, b.P) : fwd_rows(N, b.P, L)) * s_anchors[s];
            a += s_anchors[s];
            smp += s_anchors[s] * ((u32)b.P * s_cams[s] * (u32)L);
            reg += s_cams[s] * (u32)L;
        }
        b.t.anchor_start[S] = a;
        b.t.sample_start[S] = smp;
        b.t.region_start[S] = reg;
        b.t.row_start[S] = rows;
        rstart[S] = reg;
    }
    __syncthreads();
    // the XCD slots' ranges, every scene cut on its own: its first unit in each
    // slot, and (32 threads a slot) a slot's units before each scene
    auto scene_units = [&](int s) {
        const int N = (int)s_cams[s];
        const int rows = backward ? bwd_rows(N, b.P) : fwd_rows(N, b.P, L);
        return UnitGroup{1, N, (int)s_anchors[s], rows, 0, rows};
    };
    for (int i = tid; i < kSlots * S; i += blockDim.x) {
        slot_first[i] = scene_units(i % S).first(i / S);
        b.t.slot_first[i] = slot_first[i];
    }
    __syncthreads();
    {
        static_assert(kSlots * 32 == 256, "32 threads a slot");
        const int x = tid >> 5, sl = tid & 31, per = (S + 31) / 32;
        const int s0 = min(sl * per, S), s1 = min(s0 + per, S);
        auto units = [&](int s) {
            return (x + 1 < kSlots ? slot_first[(x + 1) * S + s] : scene_units(s).units()) -
                   slot_first[x * S + s];
        };
        u64 sum = 0;
        for (int s = s0; s < s1; ++s) sum += units(s);
        u64 run = sum;
#pragma unroll
        for (int d = 1; d < 32; d <<= 1) {
            const u64 t = __shfl_up(run, d, 32);
            if (sl >= d) run += t;
        }
        u64* start = b.t.slot_start + x * (S + 1);
        if (sl == 31) start[S] = run;
        run -= sum;
        for (int s = s0; s < s1; ++s) {
            start[s] = run;
            run += units(s);
        }
    }
    if (!backward) return;
    for (int s = tid; s < S; s += blockDim.x) {
        // sample / per_anchor for a sample < 2^30 as (sample * m) >> k, m = ceil(2^k / d)
        const u32 per_anchor = (u32)b.P * s_cams[s] * (u32)L;
        int lg = 0;
        while ((1u << lg) < per_anchor) ++lg;
        const int k = 32 + lg;
        b.t.magic[s] = ((1ull << k) + per_anchor - 1) / per_anchor;
        b.t.magic_shift[s] = (u32)k;
    }
    __syncthreads();

    const u32 R = rstart[S];
    // (H, W) of every region
    for (u32 g = tid; g < R; g += blockDim.x) {
        int lo = 0, hi = S - 1;                    // last scene with rstart <= g
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (rstart[mid] <= g) lo = mid; else hi = mid - 1;
        }
        const u32 i = g - rstart[lo];
        sh_h[g] = (uint16_t)b.scenes[lo].spatial_shapes[2 * i];
        sh_w[g] = (uint16_t)b.scenes[lo].spatial_shapes[2 * i + 1];
    }
    __syncthreads();

    // first cell of every region: exclusive scan of (H+1)(W+1) + 1 (the
    // bilinear cells and the region's outside cell), regions in order
    {
        const u32 per = (R + blockDim.x - 1) / blockDim.x;
        const u32 g0 = tid * per;
        u32 sum = 0;
        for (u32 k = 0; k < per; ++k)
            if (g0 + k < R) sum += ((u32)sh_h[g0 + k] + 1u) * ((u32)sh_w[g0 + k] + 1u) + 1u;
        u32 total;
        u32 run = block_inclusive_scan(sum, lds4, &total) - sum;
        for (u32 k = 0; k < per; ++k) {
            if (g0 + k < R) {
                b.t.cell_start[g0 + k] = run;
                run += ((u32)sh_h[g0 + k] + 1u) * ((u32)sh_w[g0 + k] + 1u) + 1u;
            }
        }
    }

    // the heavy cameras of scene s's level L - 1 - ld: the first ones
    auto heavy_cams = [&](int s, int ld) {
        return min(max((int)b.heavy[s] - ld * (int)s_cams[s], 0), (int)s_cams[s]);
    };
    // slot groups: (class, level descending, scene), each holding the scene's
    // cameras of the class; their first slots by a scan over all groups in that
    // order (one thread walking them took most of the kernel's 45 us for 12
    // scenes of 4 levels)
    {
        const int groups = 5 * L * S;
        auto bit = [&](const uint32_t* m, int s) { return (int)(m[s >> 5] >> (s & 31) & 1); };
        // classes: wide heavy, wide light, heavy, light, sparse light
        auto value = [&](int i, int* at) {
            const int cls = i / (L * S), rest = i - cls * (L * S), ld = rest / S, s = rest - ld * S;
            const int light = cls == 1 || cls >= 3, h = heavy_cams(s, ld);
            const bool mine = cls == (light && bit(b.thin, s) ? 4 : 2 * !bit(b.wide, s) + light);
            *at = mine ? (light * L + ld) * S + s : -1;
            return !mine ? 0u : light ? s_cams[s] - (u32)h : (u32)h;
        };
        const int per = (groups + blockDim.x - 1) / blockDim.x;
        const int i0 = tid * per, i1 = min(i0 + per, groups);
        int at;
        u32 sum = 0;
        for (int i = i0; i < i1; ++i) sum += value(i, &at);
        u32 total;
        u32 run = block_inclusive_scan(sum, lds4, &total) - sum;
        for (int i = i0; i < i1; ++i) {
            const u32 v = value(i, &at);
            if (at >= 0) grp[at] = run;
            run += v;
        }
    }
    __syncthreads();
    for (u32 g = tid; g < R; g += blockDim.x) {
        int lo = 0, hi = S - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (rstart[mid] <= g) lo = mid; else hi = mid - 1;
        }
        const int s = lo;
        const u32 i = g - rstart[s];
        const int n = (int)(i / (u32)L), l = (int)(i % (u32)L);
        const int h = heavy_cams(s, L - 1 - l), light = n >= h;
        const u32 slot = grp[(light * L + (L - 1 - l)) * S + s] + (u32)(light ? n - h : n);
        b.t.slot_scene[slot] = (u32)s;
        b.t.slot_region[slot] = i;
        tiles[slot] = (((u32)sh_h[g] + kTileH - 1) / kTileH) * (((u32)sh_w[g] + kTileW - 1) / kTileW);
    }
    __syncthreads();
    // first tile of every slot
    {
        const u32 per = (R + blockDim.x - 1) / blockDim.x;
        const u32 g0 = tid * per;
        u32 sum = 0;
        for (u32 k = 0; k < per; ++k)
            if (g0 + k < R) sum += tiles[g0 + k];
        u32 total;
        u32 run = block_inclusive_scan(sum, lds4, &total) - sum;
        for (u32 k = 0; k < per; ++k) {
            if (g0 + k < R) {
                b.t.tile_start[g0 + k] = run;
                run += tiles[g0 + k];
            }
        }
        if (tid == 0) b.t.tile_start[R] = total;
    }
}

hipError_t launch_batch_tables(const BatchArgs& b, bool backward, hipStream_t s) {
    mark_begin("batch_tables", s);
    hipLaunchKernelGGL(batch_tables_kernel, dim3(1), dim3(256), 0, s, b, backward ? 1 : 0);
    mark_end(s);
    return hipGetLastError();
}

}  // namespace msda
