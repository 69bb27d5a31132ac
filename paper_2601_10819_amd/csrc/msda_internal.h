// Internal interface between the C-ABI layer (msda_api.cpp) and the HIP
// kernels (msda_fwd.hip, msda_bwd.hip, msda_sort.hip, msda_util.hip). Not
// installed; not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/msda.h"

namespace msda {

// Byte offset used for a corner outside its level: at or beyond the end of
// every feature resource (a batch item is at most kOOB bytes, one buffer
// resource with 32-bit offsets), so a buffer load returns zeros; a lane adds
// at most one row (<= kMaxRowBytes) to it, which cannot wrap past 2^32.
constexpr uint32_t kMaxRowBytes = 4096u;
constexpr uint32_t kOOB = 0xFFFFE000u;

// ---------------------------------------------------------------- view order
//
// In view order the work of a call is cut, camera-major, into kSlots
// contiguous ranges of equal work. Range x runs on the workgroups whose index
// is x modulo kSlots: the hardware hands workgroups to the chip's kSlots XCDs
// round-robin, so a range stays on one XCD and its L2 holds the pyramids of
// the few cameras the range is working through instead of every camera's. A
// unit of work, one wave's, is one anchor over a row of cameras.
constexpr int kSlots = 8;

// A launch has fewer than 2^32 work-items; one of more waves than this goes in
// parts.
constexpr uint64_t kMaxLaunchWaves = 1u << 25, kMaxSlotUnits = kMaxLaunchWaves / kSlots;

// The units of slot x: [first[x], end[x]).
struct SlotCuts {
    uint64_t first[kSlots], end[kSlots];

    // the most of a slot
    uint64_t most() const {
        uint64_t m = 0;
        for (int x = 0; x < kSlots; ++x)
            if (end[x] - first[x] > m) m = end[x] - first[x];
        return m;
    }
    // the slots' units from the at-th on, as many as a launch takes
    SlotCuts part(uint64_t at) const {
        SlotCuts c;
        for (int x = 0; x < kSlots; ++x) {
            c.first[x] = first[x] + at < end[x] ? first[x] + at : end[x];
            c.end[x] = end[x] - c.first[x] < kMaxSlotUnits ? end[x] : c.first[x] + kMaxSlotUnits;
        }
        return c;
    }
};

// Units numbered row by row: those of B batch items of N cameras and A anchors,
// rows [row0, row0 + nrows) of `rows`, row j the cameras [N*j/rows,
// N*(j+1)/rows). They are cut into ranges of equal work, not of equal numbers
// of units: where the cameras are no multiple of the rows, rows differ in
// length, and the slots that got the long ones ended the launch (900 anchors,
// 9 cameras of 256 x 448, FP32 forward 133 -> 89 us, 12 of 512 x 704 with 5
// levels 224 -> 185). A camera of an anchor counts kCamWork and a unit by
// itself kUnitWork: 10, 17 and 25 cameras take 96, 158 and 229 us with 4 and 1,
// 103, 148 and 221 with the cameras alone; 133, 192 and 274 by units.
constexpr uint32_t kCamWork = 4, kUnitWork = 1;

struct UnitGroup {
    int B, N, A, rows, row0, nrows;
    __host__ __device__ uint64_t units() const {
        return (uint64_t)B * (uint32_t)nrows * (uint32_t)A;
    }
    // of an anchor's units in the rows before j
    __host__ __device__ uint32_t before(int j) const {
        const uint32_t cams = (uint32_t)(N * j) / (uint32_t)rows -
                              (uint32_t)(N * row0) / (uint32_t)rows;
        return kCamWork * cams + kUnitWork * (uint32_t)(j - row0);
    }
    // the first unit of slot x
    __host__ __device__ uint64_t first(int x) const {
        if (x >= kSlots) return units();
        const uint64_t item = (uint64_t)before(row0 + nrows) * (uint32_t)A;
        const uint64_t w = (uint64_t)B * item / kSlots * (uint32_t)x;
        if (w == 0) return 0;
        const uint64_t b = B == 1 ? 0 : w / item, in = w - b * item;
        int lo = row0, hi = row0 + nrows - 1;       // the last row with no more than `in` before it
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if ((uint64_t)before(mid) * (uint32_t)A <= in) lo = mid; else hi = mid - 1;
        }
        const uint64_t left = in - (uint64_t)before(lo) * (uint32_t)A;
        const uint32_t unit = before(lo + 1) - before(lo);
        return (b * (uint32_t)nrows + (uint32_t)(lo - row0)) * (uint32_t)A +
               (left + unit - 1) / unit;
    }
    SlotCuts cuts() const {
        SlotCuts c;
        for (int x = 0; x < kSlots; ++x) {
            c.first[x] = first(x);
            c.end[x] = first(x + 1);
        }
        return c;
    }
};

// Workgroups of `waves` waves for `most` units in every slot (a launch's share
// of them).
inline unsigned slot_blocks(uint64_t most, int waves) {
    if (most > kMaxSlotUnits) most = kMaxSlotUnits;
    return (unsigned)(kSlots * ((most + (uint64_t)waves - 1) / (uint64_t)waves));
}

// The forward: partial row j of a batch item with N cameras
// covers cameras [N*j/rows, N*(j+1)/rows), and one wave sums one anchor over
// one row. Rows are as short as the workspace's 8 rows per batch item allow
// to grow: one camera for a multiple of 8 up to 64 cameras (a wave per camera
// took 0.325 ms at the 64-camera scene in BF16, 2 cameras 0.332, 4 0.366, 8
// 0.385; FP32 0.577, 0.649, 0.752), and at most 64 rows so that the
// workspace stays bounded (max_fwd_rows). Where a camera has few samples,
// rather as many cameras as hold kMinRowSamples: a wave stages 64 samples at a
// time, and every row is written and read once more. 49 cameras of 7 x 3
// samples 70 -> 50 us, 63 of 7 x 4 45 -> 35, 26 of 11 x 4 173 -> 159, 53 of 11
// x 4 355 -> 343 (with 32 samples 57, 35, 176, 348); 13 x 4 are a row.
constexpr int kMinFwdRows = 8, kMaxFwdRows = 64, kMinRowSamples = 48;

__host__ __device__ inline int max_fwd_rows(int N) {
    return N < kMinFwdRows ? N : N >= kMaxFwdRows ? kMaxFwdRows : N / 8 * 8;
}

__host__ __device__ inline int fwd_rows(int N, int P, int L) {
    const int rows = max_fwd_rows(N), cams = (kMinRowSamples + P * L - 1) / (P * L);
    const int few = ((N + cams - 1) / cams + 7) / 8 * 8;
    return few < rows ? few : rows;
}

// The backward, whose rows need no combining: one camera per row, or as many
// as hold kMinRowPairs pairs where anchors have few keypoints, and a wave's start
// is most of its work (64 cameras of 256 x 448, 900 anchors, BF16, rows of 1 / 4 /
// 7 / 13 / 26 pairs at least: 1 keypoint, 4 levels 69 / 37 / 41 / 44 / 42 us, 1
// level 54 / 22 / 22 / 21 / 21; 4 keypoints 127 / 127 / 123 / 128 / 136 and 70 / 70
// / 55 / 52 / 53; 6 keypoints 180 / 180 / 178 / 186 / 196 and 87 / 87 / 72 / 72 / 74.
// 16 cameras FP32, 6 keypoints 71 / 71 / 80 / 85 / 80: there the longer rows end
// the launch, and a line that suits both is not in sight).
constexpr int kMinRowPairs = 7;

__host__ __device__ inline int bwd_rows(int N, int P) {
    const int cams = P >= kMinRowPairs ? 1 : (kMinRowPairs + P - 1) / P;
    return (N + cams - 1) / cams;
}

// Everything one forward/backward launch needs. Pointers are device memory.
struct OpArgs {
    const void* feat;             // [B][R][C], dtype below
    const int32_t* shapes;        // [N][L][2] (H, W)
    const int32_t* starts;        // [N][L]
    const float* loc;             // [B][A][P][N][2]
    const float* w;               // [B][A][P][N][L][G]
    const float* level_scale;     // [L] (FP8) or nullptr
    const float* grad_out;        // [B][A][C] (backward)
    float* out;                   // [B][A][C] (forward)
    float* gfeat_acc;             // atomic grad_feat: FP32 [B][R][C] accumulator, or nullptr
    uint32_t* rec_key;            // sorted grad_feat: [S] bilinear-cell keys, or nullptr
    float2* rec_frac;             // sorted grad_feat: [S] (lx, ly) bilinear fractions
    const uint32_t* cell_start;   // [N*L] first cell of each region (sorted grad_feat)
    uint32_t cells_per_item;      // cells of one batch item: sum of (H+1)(W+1)
    uint32_t cell_offset;         // added to every cell key (a scene's place in a batch)
    uint32_t no_cell;             // key of a sample outside its level (sorts last)
    uint32_t sample_offset;       // added to every record index
    float* grad_loc;              // or nullptr
    float* grad_w;                // or nullptr
    const float2* wstats;         // forward: w holds logits; per (b, a, g) (max, 1/sum of exp)
    int32_t w_bf16;               // forward: w holds bfloat16 bit patterns
    int32_t B, N, L, A, P, C, G;
    int64_t R;
    uint32_t batch_bytes;         // R * C * sizeof(feat element) (<= kOOB, under 4 GiB)
    int32_t lps_shift;            // log2(lanes per sample) = log2(C / chans_per_lane)
    // Bucketed records (dense single call): 0, or A*P -- the record of
    // sample (b, a, p, n, l) then goes to bucket (b, n, l) at a*P + p, its
    // key the local cell of region (n, l) (see launch_bucket_sort).
    uint32_t rec_bucket_ap;
};

// The tiled grad_feat reduction over records sorted by bilinear cell.
// Tiles are kTileH x kTileW pixels of one region; processing slot o covers camera
// o % N at level L - 1 - o / N: coarse levels first.
constexpr int kTileH = 4, kTileW = 4;

struct TileArgs {
    const uint32_t* vals;         // sample indices, sorted by cell (stable)
    const uint32_t* off;          // [B * cells_per_item + 1] first record of each cell
    const float2* frac;           // [S] (lx, ly)
    const float* w;               // weights, [S][G]
    const float* grad_out;        // [B*A][C]
    void* grad_feat;              // [B][R][C], FP32 or BF16
    const int32_t* shapes;        // [N*L][2]
    const int32_t* starts;        // [N*L]
    const uint32_t* cell_start;   // [N*L]
    const uint32_t* tile_start;   // [N*L + 1], by processing slot
    const float* view_scale;      // [B*A][N] per-view weight factor (fused form), or nullptr
    int32_t N, L;                 // cameras and levels (to find a sample's view)
    // the tiles of each batch item (slot order) to reduce: [tile_begin,
    // tile_split) coarse (all waves of a block each), [tile_split, tile_end)
    // light (one wave each)
    uint32_t tile_begin, tile_split, tile_end;
    int32_t block_waves;          // waves per block, 4 or 8
    int32_t sparse;               // 0, or the sparse light tiles a wave takes, one per sub-wave
    uint32_t cells_per_item;
    uint32_t nrec;                // S (records, one per sample)
    int32_t NL, B, C, G;
    int64_t R;
    int32_t lps_shift;            // log2(C / chans_per_lane)
    uint64_t magic;               // sample -> anchor: s / (P*N*L) == (s * magic) >> magic_shift
    int32_t magic_shift;
};

// Batched form: tables over all scenes, built on the device from the scene
// table by batch_tables_kernel. Regions are numbered scene by scene (scene
// s owns regions [region_start[s], region_start[s+1]), camera-major); slots
// order the regions for the tiled reduction: the scenes whose coarse tiles
// take 8 waves (a launch of their own) before the others, heavy (coarse)
// levels first, then by level (coarsest first), scene and camera; sparse light
// tiles of all scenes (a launch of their own, too) last.
constexpr int kMaxBatchScenes = 256;
constexpr int kMaxBatchRegions = 4096;

struct BatchTables {
    uint32_t* anchor_start;       // [S+1] first anchor (over all scenes) of each scene
    uint32_t* sample_start;       // [S+1] first sample / record of each scene
    uint32_t* region_start;       // [S+1] first region of each scene
    uint64_t* row_start;          // [S+1] first view-order unit of each scene
    uint64_t* slot_start;         // [kSlots][S+1] a slot's units before each scene
    uint64_t* slot_first;         // [kSlots][S] the scene's first unit in the slot
    uint32_t* cell_start;         // [regions] first cell of each region (global)
    uint32_t* slot_scene;         // [regions] scene of each slot
    uint32_t* slot_region;        // [regions] region (within its scene) of each slot
    uint32_t* tile_start;         // [regions + 1] first tile of each slot
    uint64_t* magic;              // [S] sample -> anchor division by P*Ncam*L
    uint32_t* magic_shift;        // [S]
};

struct BatchArgs {
    const msda_scene* scenes;     // device scene table
    int32_t S, L, P, C, G;
    const float* level_scale;
    BatchTables t;
    uint32_t total_anchors;
    uint64_t slot_units;          // view-order units of all scenes in a slot, at most
    uint64_t slot_begin;          // the first of them in this launch
    uint32_t total_samples;
    uint32_t total_cells;
    uint32_t total_regions;
    int32_t lps_shift;            // log2(C / chans_per_lane)
    uint32_t* rec_key;            // backward, grad_feat records (or nullptr)
    float2* rec_frac;
    int32_t rec_bucketed;         // records written per (scene, region) bucket (launch_bucket_sort_batched)
    // weight flags: forward, softmax statistics of every anchor (scenes in
    // order; w holds logits) and BF16 weights; backward, FP32 weights of
    // every sample (scenes in order), read in place of each scene's weights
    const float2* wstats;
    int32_t w_bf16;
    const float* w32;
    // tiled reduction
    const uint32_t* vals;
    const uint32_t* off;
    uint32_t tile_begin, tile_split, tile_end;  // as TileArgs
    int32_t block_waves;
    int32_t sparse;
    uint32_t wide[kMaxBatchScenes / 32];   // bit s: scene s's coarse tiles take 8 waves
    uint32_t thin[kMaxBatchScenes / 32];   // bit s: scene s's light tiles are sparse
    uint16_t heavy[kMaxBatchScenes];       // scene s's heavy (coarse) regions
};

enum FeatType { kF32 = 0, kBF16 = 1, kFP8 = 2, kF16 = 3 };

// Keypoint projection (device pointers).
struct ProjArgs {
    const float* anchors;         // [B][A][10] x, y, z, w, l, h, yaw, vx, vy, vz
    const float* keypoints;       // [B][A][P][3] box-frame offsets in units of (w, l, h)
    const float* projection;      // [B][N][3][4]
    const int32_t* image_hw;      // [N][2] (H, W) pixels
    float* loc;                   // [B][A][P][N][2]
    uint8_t* visible;             // [B][A][N]
    int32_t B, A, P, N;
    float dt;
};

// LDS of a forward wave's staging of `chunk` samples: each sample's 4 corner
// offsets and, per channel group, its 4 corner weights times the group's
// weight; with more groups than kPackedGroups the corner weights once and the
// groups' weights beside them (16 cameras of 256 x 448, 900 anchors, FP32, with
// the product per group: 16 groups 160 us, 32 245, 64 500; apart 132, 143, 178).
constexpr int kPackedGroups = 8;

__host__ __device__ constexpr size_t row_lds_bytes(int chunk, int G) {
    return (size_t)chunk * (G <= kPackedGroups ? 16 + 16 * (size_t)G : 32 + 4 * (size_t)G);
}

// Samples a wave of the forward stages at a time: 64 while `waves` waves'
// staging fits 64 KiB, else the largest power of two that does. At least 64 /
// lanes per sample, since G is at most the lanes per sample.
inline int fwd_chunk_samples(int waves, int G) {
    int c = 64;
    while (c > 1 && (size_t)waves * row_lds_bytes(c, G) > 65536) c /= 2;
    return c;
}
// Launchers return hipSuccess or the launch error. They enqueue only.
hipError_t launch_forward(const OpArgs& a, int dtype, int cpl, int waves, hipStream_t s);
hipError_t launch_backward(const OpArgs& a, int dtype, int cpl, int waves, hipStream_t s);
// View order: `waves` waves per workgroup, each its own unit. The forward
// writes partial rows to part and adds them into out in row order, part_rows
// (>= min(fwd_rows, kMinFwdRows)) rows [B][part_rows][A][C] FP32 at a
// time; the sums do not depend on part_rows.
hipError_t launch_forward_view(const OpArgs& a, int dtype, int cpl, int waves, int part_rows,
                               float* part, hipStream_t s);
hipError_t launch_backward_view(const OpArgs& a, int dtype, int cpl, int waves, hipStream_t s);
hipError_t launch_gfeat_tiles(const TileArgs& t, int out_dtype, int cpl, hipStream_t s);
// cell_start[N*L] and tile_start[N*L + 1] from the shapes.
hipError_t launch_region_tables(const int32_t* shapes, int32_t N, int32_t L, uint32_t* cell_start,
                                uint32_t* tile_start, hipStream_t s);
// Stable sort of the n record keys (keys_a; values = the indices, or the
// caller's in vals_a when vals_given) by key in [0, nrows]; *sorted_vals
// receives the sorted values (in vals_a or vals_b) and off[0..nrows] the
// segment starts. n_dev (or nullptr): a device count that caps n at run
// time. scratch: sort_scratch_words(n) words.
hipError_t launch_sort_records(uint32_t* keys_a, uint32_t* keys_b, uint32_t* vals_a,
                               uint32_t* vals_b, uint32_t n, uint32_t nrows, uint32_t* scratch,
                               uint32_t* off, uint32_t** sorted_vals, hipStream_t s,
                               const uint32_t* n_dev = nullptr, bool vals_given = false);
size_t sort_scratch_words(uint32_t n);
// The dense single call's record sort, one workgroup per bucket (b, region):
// bucket k = b*N*L + r holds the A*P records of region r of batch item b in
// (anchor, keypoint) order at [k*ap, (k+1)*ap) of keys, key = the local cell
// in [0, (H+1)(W+1)] ((H+1)(W+1): outside the level). Sorts each bucket by
// key, stably, in LDS; writes vals[k*ap + i] = the sample index of the
// bucket's i-th record in key order and off[] of the bucket's cells (global
// cell b*cells_per_item + cell_start[r] + local), and off[B*cells_per_item]
// = B*N*L*ap. Also writes the region tables of launch_region_tables
// (cell_start, tile_start). Requires ap <= kBucketMaxRecords,
// (H+1)(W+1) + 1 <= kBucketMaxKeys for every region, N*L <= 1024, and
// bucket_sort_lds_bytes(ap) of LDS. The visible-view form (place, items
// non-null: the exclusive scan of the visible flags over the view-major items
// (b*N + n)*A + a and the compacted item list): bucket (b, n, l) holds the
// cnt*P records of the cnt visible anchors of (b, n), at s0*P*L + l*cnt*P
// with s0 = place[(b*N + n)*A], in (anchor, keypoint) order, ap = A*P
// bounding cnt*P; vals and off as above, off[B*cells_per_item] = the number
// of visible records.
constexpr uint32_t kBucketMaxRecords = 1u << 15;
constexpr uint32_t kBucketMaxKeys = 1u << 17;
size_t bucket_sort_lds_bytes(uint32_t ap);
hipError_t launch_bucket_sort(const uint32_t* keys, const int32_t* shapes, int32_t B, int32_t N,
                              int32_t L, int32_t A, int32_t P, uint32_t cells_per_item,
                              uint32_t* vals, uint32_t* off, uint32_t* cell_start,
                              uint32_t* tile_start, const uint32_t* place, const uint32_t* items,
                              hipStream_t s);
// The batched form's record sort: bucket k = the batch's region k (scene s,
// region r of it), A_s*P records at sample_start[s] + r*A_s*P, keyed by
// local cell; writes the sorted global sample indices to vals (bucket k's
// part at the same place) and off[] of the batch's cells (cell_start of the
// batch tables, (H+1)(W+1) + 1 per region), off[total_cells] = total
// samples. max_ap: the largest A_s*P (<= kBucketMaxRecords; LDS
// bucket_sort_lds_bytes(max_ap)).
hipError_t launch_bucket_sort_batched(const BatchArgs& b, uint32_t max_ap, uint32_t* vals,
                                      uint32_t* off, hipStream_t s);

// Keypoint projection and the visible-view form (msda_vis.hip).
hipError_t launch_project_keypoints(const ProjArgs& p, hipStream_t s);
// place[0..V] = exclusive scan of the view-major visibility flags (place[V]
// = the number of visible items), items[place[v]] = v, and *rec_count =
// place[V] * per_item (or nothing when rec_count is nullptr); partial:
// visible_partial_words(V) words. V = B * N * A > 0.
size_t visible_partial_words(size_t V);
hipError_t launch_visible_items(const uint8_t* visible, int B, int N, int A, uint32_t per_item,
                                uint32_t* place, uint32_t* items, uint32_t* rec_count,
                                uint32_t* partial, hipStream_t s);
// vt (or nullptr): the fused form's per-view weights [B][A][N].
hipError_t launch_forward_visible(const OpArgs& a, int dtype, int cpl, int waves,
                                  const uint32_t* items, const uint32_t* count,
                                  const uint32_t* place, const uint8_t* visible, const float* vt,
                                  float* part, hipStream_t s);
// item_dot (or nullptr): per item, <grad_out, the anchor's feature in the view>.
hipError_t launch_backward_visible(const OpArgs& a, int dtype, int cpl, int waves,
                                   const uint32_t* items, const uint32_t* place,
                                   const uint32_t* count, uint32_t* rec_val, const float* vt,
                                   float* item_dot, hipStream_t s);
// Fused weight generation (per-group softmax of logits, BF16 weights).
// stats[(b*A + a)*G + g] = (max, 1 / sum of exp(logit - max)) over the
// anchor's P*N*L logits of group g, and the softmax weights of all BA*PNL*G
// entries, FP32; either may be nullptr. Logits FP32 or bfloat16 bit patterns.
// scratch: softmax_scratch_bytes, used (if given) for weights alone.
size_t softmax_scratch_bytes(int64_t BA, size_t n, int G);    // n = PNL*G
hipError_t launch_softmax(const void* logits, bool bf16, int BA, int PNL, int G, float2* stats,
                          float* weights, float2* scratch, hipStream_t s);
// w[i] = the bfloat16 weight src[i], widened, for all BA*PNL*G entries.
hipError_t launch_weights_f32(const void* src, int BA, int PNL, int G, float* w, hipStream_t s);
// In place: grad[i] = w[i] * (grad[i] - sum over the anchor's group of w * grad),
// the gradient through the per-group softmax. scratch: as for launch_softmax.
hipError_t launch_softmax_grad(const float* w, float* grad, int BA, int PNL, int G, float2* scratch,
                               hipStream_t s);
hipError_t launch_view_scale(const uint8_t* visible, const float* score, int BA, int N,
                             float* vt, hipStream_t s);
hipError_t launch_grad_score(const float* grad_out, const float* out, const uint8_t* visible,
                             const float* score, const uint32_t* place, const float* item_dot,
                             int B, int A, int N, int C, float* grad_score, hipStream_t s);
int sort_passes(uint32_t max_key);

hipError_t launch_batch_tables(const BatchArgs& b, bool backward, hipStream_t s);
hipError_t launch_forward_batched(const BatchArgs& b, int dtype, int cpl, int waves, int blocks,
                                  hipStream_t s);
hipError_t launch_backward_batched(const BatchArgs& b, int dtype, int cpl, int waves, int blocks,
                                   hipStream_t s);
// Batched gathers in view order: one wave per unit of every scene, scenes in
// order. The forward's partial rows go to part ([units][C] FP32) and are
// added into each scene's out.
hipError_t launch_forward_batched_view(const BatchArgs& b, int dtype, int cpl, int waves,
                                       float* part, hipStream_t s);
hipError_t launch_backward_batched_view(const BatchArgs& b, int dtype, int cpl, int waves,
                                        hipStream_t s);
hipError_t launch_gfeat_tiles_batched(const BatchArgs& b, int out_dtype, int cpl, hipStream_t s);

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);
hipError_t launch_f32_to_bf16(const float* src, uint16_t* dst, size_t n, hipStream_t s);
hipError_t launch_f32_to_f16(const float* src, uint16_t* dst, size_t n, hipStream_t s);
// max_region_rows: the largest H*W over the regions (sizes the grid).
hipError_t launch_quantize_fp8(const float* x, const int32_t* shapes, const int32_t* starts,
                               int32_t B, int32_t N, int32_t L, int64_t R, int32_t C,
                               int64_t max_region_rows, uint8_t* codes, float* level_scale,
                               uint32_t* amax_ws, hipStream_t s);
hipError_t launch_stream_copy(void* dst, const void* src, size_t bytes, hipStream_t s);

// The most LDS a gather's workgroup of `waves` waves takes.
size_t gather_lds_bytes(int waves, int C, int G);

// The least workspace msda_forward_ws takes for d: kMinFwdRows partial rows
// per batch item in view order, where msda_forward_workspace_size has room for all.
size_t forward_min_workspace(const msda_desc* d);

// Sets the thread's last-error message (msda_last_error) and returns st.
msda_status set_error(msda_status st, const char* message);

// Benchmark instrumentation (msda_set_kernel_events): called around every
// kernel launch; records the caller's events when enabled, else does nothing.
void mark_begin(const char* kernel, hipStream_t s);
void mark_end(hipStream_t s);

}  // namespace msda
