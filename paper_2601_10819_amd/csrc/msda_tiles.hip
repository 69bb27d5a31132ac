// The deterministic grad_feat reduction of the backward, after the
// samples' records are sorted by bilinear cell (msda_sort.hip): each 4x4 tile
// of pixels of a region visits the 5x5 cells whose samples touch it, in a
// fixed order, and adds w * cw * grad_out[anchor] of each sample's corners
// that fall in the tile to register accumulators; each sample's grad_out row
// is read once per tile it touches (about 1.6 times on average) instead of
// once per corner. The tile's records are split between its waves and the
// partial sums added in a fixed order, so grad_feat is bitwise reproducible;
// every pixel is written once, in FP32, BF16 or FP16 (rounded to nearest
// even), zeros where no sample lands.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "msda_common.h"

namespace msda {

template <int I>
using int_c = std::integral_constant<int, I>;

// f(int_c<0>{}), ..., f(int_c<N-1>{}): a loop whose index is a compile-time constant.
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(int_c<I>{});
        static_for<N, I + 1>(f);
    }
}

template <class OT, int CPL>
__device__ __forceinline__ void store_row(void* base, size_t elem, const float* acc) {
    if constexpr (OT::kBytes == 4) {
        float* p = static_cast<float*>(base) + elem;
        if constexpr (CPL == 4) {
            *reinterpret_cast<float4*>(p) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        } else {
#pragma unroll
            for (int i = 0; i < CPL; ++i) p[i] = acc[i];
        }
    } else {
        // one rounding of the FP32 sum to the storage type
        auto rnd = [](float x) -> u32 {
            if constexpr (OT::kKind == 3) return f16_rne(x);
            else return bf16_rne(x);
        };
        uint16_t* p = static_cast<uint16_t*>(base) + elem;
        if constexpr (CPL == 4) {
            u32 lo, hi;
            if constexpr (OT::kKind == 3) {
                lo = rnd(acc[0]) | (rnd(acc[1]) << 16);
                hi = rnd(acc[2]) | (rnd(acc[3]) << 16);
            } else {
                lo = bf16x2_rne(acc[0], acc[1]);
                hi = bf16x2_rne(acc[2], acc[3]);
            }
            *reinterpret_cast<u32x2*>(p) = u32x2{lo, hi};
        } else {
#pragma unroll
            for (int i = 0; i < CPL; ++i) p[i] = (uint16_t)rnd(acc[i]);
        }
    }
}

template <int CPL>
__device__ __forceinline__ void load_go(const float* p, float* v) {
    if constexpr (CPL == 4) {
        const float4 t = *reinterpret_cast<const float4*>(p);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else {
#pragma unroll
        for (int i = 0; i < CPL; ++i) v[i] = p[i];
    }
}

// Tables of the tiled reduction for one batch item, from the shapes: the
// first cell of each region (regions in order, (H+1)(W+1) bilinear cells
// each and one for the region's samples outside the level) and the first tile
// of each processing slot (coarse levels first: slot o = (L-1-l)*N + n). One
// block of 256 threads; N*L <= 1024 regions, 4 per thread.
__global__ void __launch_bounds__(256) region_tables_kernel(const int32_t* shapes, int N, int L,
                                                            u32* cell_start, u32* tile_start) {
    __shared__ u32 lds4[4];
    const int NL = N * L;
    u32 cells[4], tiles[4], sum_c = 0, sum_t = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = 4 * threadIdx.x + k;
        cells[k] = tiles[k] = 0u;
        if (i < NL) {
            const u32 H = (u32)shapes[2 * i], W = (u32)shapes[2 * i + 1];
            cells[k] = (H + 1) * (W + 1) + 1;    // + the region's outside cell
            const int o = i;                     // slot o -> region r
            const int r = (o % N) * L + (L - 1 - o / N);
            const u32 Hr = (u32)shapes[2 * r], Wr = (u32)shapes[2 * r + 1];
            tiles[k] = ((Hr + kTileH - 1) / kTileH) * ((Wr + kTileW - 1) / kTileW);
        }
        sum_c += cells[k];
        sum_t += tiles[k];
    }
    u32 total_c, total_t;
    u32 run_c = block_inclusive_scan(sum_c, lds4, &total_c) - sum_c;
    u32 run_t = block_inclusive_scan(sum_t, lds4, &total_t) - sum_t;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = 4 * threadIdx.x + k;
        if (i < NL) {
            cell_start[i] = run_c;
            tile_start[i] = run_t;
        }
        run_c += cells[k];
        run_t += tiles[k];
    }
    if (threadIdx.x == 0) tile_start[NL] = total_t;
}

// One sample's corners that fall in the tile, added to the accumulators.
// The sample's cell sits at tile offset (DY, DX), so the corner -> pixel map
// is static: corners land on (DY-1, DX-1), (DY-1, DX), (DY, DX-1), (DY, DX).
// f holds the bilinear factors ((1-ly)(1-lx), (1-ly)lx, ly(1-lx), ly lx),
// computed once per record; each corner's weight is its factor times wv.
template <int DY, int DX, int TH, int TW, int CPL>
__device__ __forceinline__ void add_sample(float (&acc)[TH][TW][CPL], float4 f, float wv,
                                           const float* gv) {
    const float k00 = f.x * wv, k01 = f.y * wv;
    const float k10 = f.z * wv, k11 = f.w * wv;
    if constexpr (DY >= 1 && DX >= 1) {
#pragma unroll
        for (int i = 0; i < CPL; ++i) acc[DY - 1][DX - 1][i] = fmaf(k00, gv[i], acc[DY - 1][DX - 1][i]);
    }
    if constexpr (DY >= 1 && DX < TW) {
#pragma unroll
        for (int i = 0; i < CPL; ++i) acc[DY - 1][DX][i] = fmaf(k01, gv[i], acc[DY - 1][DX][i]);
    }
    if constexpr (DY < TH && DX >= 1) {
#pragma unroll
        for (int i = 0; i < CPL; ++i) acc[DY][DX - 1][i] = fmaf(k10, gv[i], acc[DY][DX - 1][i]);
    }
    if constexpr (DY < TH && DX < TW) {
#pragma unroll
        for (int i = 0; i < CPL; ++i) acc[DY][DX][i] = fmaf(k11, gv[i], acc[DY][DX][i]);
    }
}

// One sample of a statically known cell (DY, DX).
template <int DY, int DX, int CPL>
__device__ __forceinline__ void cell_sample(float (&acc)[4][4][CPL], float4 f, float wv,
                                            const float* gv) {
    add_sample<DY, DX, 4, 4, CPL>(acc, f, wv, gv);
}

// One sample of the cell `at` = dy * 5 + dx, known at run time only.
template <int CPL>
__device__ __forceinline__ void add_sample_at(int at, float (&acc)[4][4][CPL], float4 f, float wv,
                                              const float* gv) {
#define MSDA_CELL(P) \
    case P: add_sample<(P) / 5, (P) % 5, 4, 4, CPL>(acc, f, wv, gv); break;
#define MSDA_CELLS(P) \
    MSDA_CELL(P) MSDA_CELL(P + 1) MSDA_CELL(P + 2) MSDA_CELL(P + 3) MSDA_CELL(P + 4)
    switch (at) {
        MSDA_CELLS(0) MSDA_CELLS(5) MSDA_CELLS(10) MSDA_CELLS(15) MSDA_CELLS(20)
        default: break;
    }
#undef MSDA_CELLS
#undef MSDA_CELL
}

// Floats per record-table entry: the 4 bilinear factors, the anchor, the cell
// (sparse tiles), 2 spare, then the G weights (16-byte multiple, so the factors load as one
// vector).
__host__ __device__ inline int tile_entry_floats(int G) { return 8 + ((G + 3) & ~3); }

// Floats of a wave's LDS with sparse tiles: the record table and each sub-wave's
// cell boundaries.
__host__ __device__ inline int sparse_wave_floats(int lps_shift, int G) {
    const int bounds = (64 >> lps_shift) * (kTileH + 1) * (kTileW + 2);
    return 64 * tile_entry_floats(G) + ((bounds + 3) & ~3);
}

// Records of a sparse tile whose grad_out rows are loaded together.
constexpr int kSparseRows = 4;

// Everything one tile's reduction needs (from the single-call or the
// batched tables).
struct TileView {
    const u32* vals;            // sorted record indices (global sample indices)
    const u32* off;             // first record of each cell
    const float2* frac;         // per record (global index): (lx, ly)
    const float* w;             // the scene's weights [S][G]
    const float* grad_out;      // the scene's grad_out [A][C]
    void* grad_feat;            // the scene's grad_feat
    size_t row_base;            // first grad_feat row of the tile's batch item
    u32 nrec;                   // records in the sort (all scenes)
    u32 sample_offset;          // first record index of the scene
    u32 sample_count;           // records of the scene
    u32 cbase;                  // first cell of the tile's region
    int H, W, start;            // the region
    int ty, tx;                 // the tile's first pixel
    int C, G;
    u64 magic;                  // scene-local sample -> anchor
    int magic_shift;
    const float* vscale;        // [anchor][N] per-view weight factor, or nullptr
    int N, L;
    bool active;
    bool w16;                   // G % 4 == 0 and w 16-byte aligned
};

// Lane i's value (i uniform) as a uniform one.
__device__ __forceinline__ u32 lane_value(u32 x, int i) {
    return (u32)__builtin_amdgcn_readlane((int)x, i);
}

// grad_out row of a whole-wave record: with a uniform anchor the row address
// is scalar arithmetic and each lane adds only its channel offset.
__device__ __forceinline__ const float* go_row(const TileView& v, u32 anchor) {
    return v.grad_out + (size_t)anchor * (u32)v.C;
}

// The table entry of the record at sorted position e; returns its anchor.
__device__ __forceinline__ u32 fill_entry(const TileView& v, u32 e, float* ent) {
    const u32 s = min(v.vals[e], v.nrec - 1u);
    const float2 fr = v.frac[s];
    // the scene-local sample (clamped into the scene: an inconsistent sort could
    // only give wrong sums, never a read outside it)
    const u32 ls = s - v.sample_offset < v.sample_count ? s - v.sample_offset : 0u;
    const float* ws = v.w + (size_t)ls * v.G;
    const u32 an = fast_div(ls, v.magic, v.magic_shift);
    if (v.vscale) {
        // the fused form: the sample's weights times its view's factor
        const u32 n = (ls / (u32)v.L) % (u32)v.N;
        const float sc = v.vscale[(size_t)an * v.N + n];
        for (int k = 0; k < v.G; ++k) ent[8 + k] = ws[k] * sc;
    } else if (v.w16) {
        // rows of G % 4 == 0 floats from a 16-byte aligned base: 16-byte loads
        // and LDS stores
        const float4* ws4 = reinterpret_cast<const float4*>(ws);
        float4* e4 = reinterpret_cast<float4*>(ent + 8);
        for (int k = 0; k < (v.G >> 2); ++k) e4[k] = ws4[k];
    } else {
        for (int k = 0; k < v.G; ++k) ent[8 + k] = ws[k];
    }
    const float hx = 1.f - fr.x, hy = 1.f - fr.y;
    *reinterpret_cast<float4*>(ent) = make_float4(hy * hx, hy * fr.x, fr.y * hx, fr.y * fr.x);
    ent[4] = __uint_as_float(an);
    return an;
}

// The reduction of one tile by `waves` waves of the block that share its
// records, this wave being the wt-th of them (waves == 1: wt == 0, and the
// other waves of the block reduce tiles of their own).
//
// A record takes 1 << lps_shift lanes (C / CPL), so a wave walks 64 >>
// lps_shift records of a cell at a time, one per sub-wave (WHOLE: lps_shift
// is 6). Each chunk's records are walked cell by cell in a static loop over
// the tile's 5x5 cells, so every record's corner -> pixel map is a
// compile-time constant (no per-record dispatch); records of a cell are
// consecutive in the sorted order. QB: records of a sub-wave whose grad_out
// rows are loaded together.
template <class OT, int CPL, bool WHOLE, int QB>
__device__ __forceinline__ void tile_reduce(const TileView& v, const int lps_shift,
                                            const int waves, const int wt, float* work) {
    constexpr int TH = kTileH, TW = kTileW;
    constexpr bool FIRST = WHOLE && QB == 2;
    // the wave index is uniform: chunk bounds and cell runs below stay scalar
    const int lane = threadIdx.x & 63, wave = uniform((int)(threadIdx.x >> 6));
    const int spw = WHOLE ? 1 : 64 >> lps_shift;            // sub-waves
    const int sub = WHOLE ? 0 : lane >> lps_shift;
    const int sl = WHOLE ? lane : lane & ((1 << lps_shift) - 1);
    const int stride = tile_entry_floats(v.G);      // floats per record-table entry
    float* tab = work + (size_t)wave * 64 * stride;
    const bool active = v.active;
    const int H = v.H, W = v.W, ty = v.ty, tx = v.tx;
    const u32 cbase = v.cbase;
    const int c0 = sl * CPL;
    const int g = c0 / (v.C / v.G);

    // The tile's cells are TH+1 rows of TW+1 consecutive cells; each row's
    // records are one contiguous range of the sorted order. Lane k holds
    // boundary k of those rows, TW+2 per row.
    static_assert((TH + 1) * (TW + 2) <= 64, "one boundary per lane");
    u32 bound = 0u;
    if (lane < (TH + 1) * (TW + 2)) {
        const int dy = lane / (TW + 2), dx = lane % (TW + 2);
        if (active && ty + dy <= H) {
            // cells past W+1 clamp to the row's end
            const u32 cell = cbase + (u32)(ty + dy) * (u32)(W + 1) + (u32)min(tx + dx, W + 1);
            bound = min(v.off[cell], v.nrec);
        }
    }
    // a row's first record and number of records (none past the region: the
    // boundaries are all 0 there)
    auto row_start = [&](int dy) { return lane_value(bound, dy * (TW + 2)); };
    auto row_len = [&](int dy) {
        const u32 a0 = row_start(dy), a1 = lane_value(bound, dy * (TW + 2) + TW + 1);
        return a1 > a0 ? a1 - a0 : 0u;
    };
    u32 total = 0;
#pragma unroll
    for (int dy = 0; dy <= TH; ++dy) total += row_len(dy);

    float acc[TH][TW][CPL];
#pragma unroll
    for (int py = 0; py < TH; ++py)
#pragma unroll
        for (int px = 0; px < TW; ++px)
#pragma unroll
            for (int i = 0; i < CPL; ++i) acc[py][px][i] = 0.f;

    // The tile's records as one flat list, in chunks of 64; chunk k goes to
    // wave k % waves. Each lane fills one table entry (all the chunk's loads
    // in flight together), then the wave walks the chunk.
    for (u32 base = (u32)(wt * 64); base < total; base += (u32)(waves * 64)) {
        const int n = (int)min(64u, total - base);
        // the boundaries are read from the lanes again in every chunk: kept
        // over the loop they take the scalar registers of everything else
        asm("" : "+v"(bound));
        u32 an = 0u;                                // lane k: the anchor of the chunk's record k
        if (lane < n) {
            // flat index -> (row dy, sorted position e)
            u32 f = base + (u32)lane;
            int dy = 0;
#pragma unroll
            for (int k = 0; k < TH; ++k)
                if (dy == k && f >= row_len(k)) { f -= row_len(k); dy = k + 1; }
            u32 e = row_start(0) + f;
#pragma unroll
            for (int k = 1; k <= TH; ++k)
                if (dy == k) e = row_start(k) + f;
            an = fill_entry(v, e, tab + lane * stride);
        }
        // LDS accesses of one wave are performed in order; keep the compiler
        // from hoisting the reads above the writes
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // flat index of each row's first record, then each cell's run
        // clipped to this chunk [base, base + n)
        u32 f0 = 0;
        static_for<TH + 1>([&](auto dyc) {
            constexpr int DY = decltype(dyc)::value;
            const u32 rlen = row_len(DY);
            if (rlen) {
                const u32 rstart = row_start(DY);
                // a cell's run [lo, hi) of the chunk
                auto lo = [&](int dx) {
                    const u32 e = lane_value(bound, DY * (TW + 2) + dx);
                    return (int)max(f0 + (e - rstart), base) - (int)base;
                };
                auto hi = [&](int dx) {
                    const u32 e = lane_value(bound, DY * (TW + 2) + dx + 1);
                    return (int)min(f0 + (e - rstart), base + (u32)n) - (int)base;
                };
                float first[TW + 1][CPL];
                if constexpr (FIRST) {
#pragma unroll
                    for (int dx = 0; dx <= TW; ++dx)
                        if (lo(dx) < hi(dx))
                            load_go<CPL>(go_row(v, lane_value(an, lo(dx))) + (u32)c0, first[dx]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                static_for<TW + 1>([&](auto dxc) {
                    constexpr int DX = decltype(dxc)::value;
                    int qq = lo(DX);
                    const int qe = hi(DX);
                    if constexpr (WHOLE) {
                        if constexpr (FIRST) {
                            if (qq < qe) {
                                const float* ent = tab + qq * stride;
                                cell_sample<DY, DX, CPL>(acc,
                                                         *reinterpret_cast<const float4*>(ent),
                                                         ent[8 + g], first[DX]);
                                ++qq;
                            }
                        }
                        for (; qq + QB <= qe; qq += QB) {
                            float gv[QB][CPL];
#pragma unroll
                            for (int k = 0; k < QB; ++k)
                                load_go<CPL>(go_row(v, lane_value(an, qq + k)) + (u32)c0, gv[k]);
                            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                            for (int k = 0; k < QB; ++k) {
                                const float* ent = tab + (qq + k) * stride;
                                cell_sample<DY, DX, CPL>(
                                    acc, *reinterpret_cast<const float4*>(ent), ent[8 + g], gv[k]);
                            }
                        }
                        for (; qq < qe; ++qq) {
                            const float* ent = tab + qq * stride;
                            float gv[CPL];
                            load_go<CPL>(go_row(v, lane_value(an, qq)) + (u32)c0, gv);
                            cell_sample<DY, DX, CPL>(acc, *reinterpret_cast<const float4*>(ent),
                                                     ent[8 + g], gv);
                        }
                    } else {
                        // sub-wave s takes the run's records s, s + spw, ...;
                        // past the run's end it loads its last record's row
                        // again and adds nothing
                        for (; qq < qe; qq += QB * spw) {
                            float gv[QB][CPL];
                            const float* ent[QB];
#pragma unroll
                            for (int k = 0; k < QB; ++k) {
                                ent[k] = tab + min(qq + k * spw + sub, qe - 1) * stride;
                                load_go<CPL>(v.grad_out +
                                                 (size_t)__float_as_uint(ent[k][4]) * v.C + c0,
                                             gv[k]);
                            }
#pragma unroll
                            for (int k = 0; k < QB; ++k)
                                if (qq + k * spw + sub < qe)
                                    cell_sample<DY, DX, CPL>(
                                        acc, *reinterpret_cast<const float4*>(ent[k]),
                                        ent[k][8 + g], gv[k]);
                        }
                    }
                });
            }
            f0 += rlen;
        });
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }

    // partial sums of the waves, added pairwise in a fixed tree order:
    // wave w += wave w + h for h = waves/2, waves/4, ..., 1
    if (waves > 1) {
        constexpr int E = TH * TW * CPL;
        float* part = work;
        __syncthreads();                             // record tables are dead from here on
        for (int h = waves >> 1; h >= 1; h >>= 1) {
            if (wt >= h && wt < 2 * h) {
#pragma unroll
                for (int py = 0; py < TH; ++py)
#pragma unroll
                    for (int px = 0; px < TW; ++px)
#pragma unroll
                        for (int i = 0; i < CPL; ++i)
                            part[((wt - h) * E + (py * TW + px) * CPL + i) * 64 + lane] =
                                acc[py][px][i];
            }
            __syncthreads();
            if (wt < h) {
#pragma unroll
                for (int py = 0; py < TH; ++py)
#pragma unroll
                    for (int px = 0; px < TW; ++px)
#pragma unroll
                        for (int i = 0; i < CPL; ++i)
                            acc[py][px][i] += part[(wt * E + (py * TW + px) * CPL + i) * 64 + lane];
            }
            __syncthreads();
        }
    }
    if (wt != 0 || !active) return;
    if constexpr (!WHOLE) {
        // the sub-waves' sums, in every sub-wave
        auto fold = [&](auto&& sum) {
#pragma unroll
            for (int py = 0; py < TH; ++py)
#pragma unroll
                for (int px = 0; px < TW; ++px)
#pragma unroll
                    for (int i = 0; i < CPL; ++i) acc[py][px][i] = sum(acc[py][px][i]);
        };
        for (int m = 1 << lps_shift; m < 8; m <<= 1)
            fold([&](float x) { return x + xor_shuffle(x, m); });
        if (lps_shift <= 3) fold([](float x) { return x + dpp<0x128>(x); });   // row_ror:8
        if (lps_shift <= 4) fold([](float x) { return swap16_sum(x); });
        fold([](float x) { return swap32_sum(x); });
    }
    const int start = v.start;
#pragma unroll
    for (int py = 0; py < TH; ++py) {
#pragma unroll
        for (int px = 0; px < TW; ++px) {
            const int y = ty + py, x = tx + px;
            // each sub-wave stores its share of the pixels
            if (y < H && x < W && (WHOLE || ((py * TW + px) & (spw - 1)) == (sub & (TH * TW - 1)))) {
                const size_t row = v.row_base + (size_t)(start + y * W + x);
                store_row<OT, CPL>(v.grad_feat, row * (size_t)v.C + (size_t)c0, acc[py][px]);
            }
        }
    }
}

// The reduction of a sparse tile by the lanes of one sub-wave (1 << lps_shift
// of them), so that a wave takes as many tiles as it has sub-waves: `v` is the
// sub-wave's tile, its records one after the other, each by a run-time dispatch
// on its cell. bnd, tab: the wave's cell boundaries and record table in LDS.
template <class OT, int CPL>
__device__ __forceinline__ void tile_reduce_sparse(const TileView& v, const int lps_shift,
                                                   u32* bnd, float* tab) {
    constexpr int TH = kTileH, TW = kTileW, NB = (TH + 1) * (TW + 2), QB = kSparseRows;
    const int lane = threadIdx.x & 63, lps = 1 << lps_shift;
    const int sub = lane >> lps_shift, sl = lane & (lps - 1);
    const int stride = tile_entry_floats(v.G);
    tab += sub * lps * stride;
    bnd += sub * NB;
    const int c0 = sl * CPL, g = c0 / (v.C / v.G);
    for (int k = sl; k < NB; k += lps) {
        const int dy = k / (TW + 2), dx = k % (TW + 2);
        u32 x = 0u;
        if (v.active && v.ty + dy <= v.H) {
            const u32 cell = v.cbase + (u32)(v.ty + dy) * (u32)(v.W + 1) +
                             (u32)min(v.tx + dx, v.W + 1);
            x = min(v.off[cell], v.nrec);
        }
        bnd[k] = x;
    }
    wave_lds_sync();
    u32 rs[TH + 1], rn[TH + 1], total = 0;          // the cell rows' first records and lengths
#pragma unroll
    for (int dy = 0; dy <= TH; ++dy) {
        rs[dy] = bnd[dy * (TW + 2)];
        const u32 end = bnd[dy * (TW + 2) + TW + 1];
        rn[dy] = end > rs[dy] ? end - rs[dy] : 0u;
        total += rn[dy];
    }
    float acc[TH][TW][CPL];
#pragma unroll
    for (int py = 0; py < TH; ++py)
#pragma unroll
        for (int px = 0; px < TW; ++px)
#pragma unroll
            for (int i = 0; i < CPL; ++i) acc[py][px][i] = 0.f;

    // the records as one flat list, a lane's entry each, lps at a time
    for (u32 base = 0; base < total; base += (u32)lps) {
        const int n = (int)min((u32)lps, total - base);
        if (sl < n) {
            u32 f = base + (u32)sl;
            int dy = 0;
#pragma unroll
            for (int k = 0; k < TH; ++k)
                if (dy == k && f >= rn[k]) { f -= rn[k]; dy = k + 1; }
            u32 e = rs[0] + f;
#pragma unroll
            for (int k = 1; k <= TH; ++k)
                if (dy == k) e = rs[k] + f;
            int dx = 0;
#pragma unroll
            for (int k = 1; k <= TW; ++k)
                if (e >= bnd[dy * (TW + 2) + k]) dx = k;
            float* ent = tab + sl * stride;
            fill_entry(v, e, ent);
            ent[5] = __int_as_float(dy * (TW + 1) + dx);
        }
        wave_lds_sync();
        for (int q = 0; q < n; q += QB) {
            float gv[QB][CPL];
#pragma unroll
            for (int k = 0; k < QB; ++k)
                load_go<CPL>(v.grad_out +
                                 (size_t)__float_as_uint(tab[min(q + k, n - 1) * stride + 4]) * v.C +
                                 c0,
                             gv[k]);
#pragma unroll
            for (int k = 0; k < QB; ++k) {
                if (q + k < n) {
                    const float* ent = tab + (q + k) * stride;
                    add_sample_at<CPL>(__float_as_int(ent[5]), acc,
                                       *reinterpret_cast<const float4*>(ent), ent[8 + g], gv[k]);
                }
            }
        }
        wave_lds_sync();
    }
    if (!v.active) return;
#pragma unroll
    for (int py = 0; py < TH; ++py) {
#pragma unroll
        for (int px = 0; px < TW; ++px) {
            const int y = v.ty + py, x = v.tx + px;
            if (y < v.H && x < v.W) {
                const size_t row = v.row_base + (size_t)(v.start + y * v.W + x);
                store_row<OT, CPL>(v.grad_feat, row * (size_t)v.C + (size_t)c0, acc[py][px]);
            }
        }
    }
}

// The last of n slots whose first tile (tile_start) is at most tt, and that
// tile. The lanes look at n / 64 apart, then at the run between: two loads in
// a row where a binary search takes one per halving (4 cameras of 128 x 224
// 89 -> 85 us, 8 cameras 46 -> 45, 6 cameras FP32 53.3 -> 52.5, 64 cameras the
// same).
__device__ __forceinline__ int slot_of(const u32* tile_start, int n, u32 tt, u32* first) {
    const int lane = threadIdx.x & 63;
    const int k = (n + 63) >> 6;
    u32 v = lane * k < n ? tile_start[lane * k] : 0xffffffffu;
    int at = (int)__popcll(__ballot(v <= tt)) - 1;      // slot 0 starts at tile 0
    int slot = at * k;
    for (int base = slot; k > 1 && base < (at + 1) * k; base += 64) {
        const int i = base + lane;
        v = i < min((at + 1) * k, n) ? tile_start[i] : 0xffffffffu;
        const int m = (int)__popcll(__ballot(v <= tt));
        if (m == 0) break;
        slot = base + m - 1;
        *first = lane_value(v, m - 1);
    }
    if (k == 1) *first = lane_value(v, at);
    return uniform(slot);
}

// The slot of tile tt, at or after slot o (which starts at *first), lane by lane.
__device__ __forceinline__ int slot_after(const u32* tile_start, int n, u32 tt, int o, u32* first) {
    for (; o + 1 < n; ++o) {
        const u32 next = tile_start[o + 1];
        if (next > tt) break;
        *first = next;
    }
    return o;
}

// The tile of id gt; ids run over batch items first, then processing slots
// within [tile_begin, tile_end). WAVE: the same id in every lane, else ids from
// the first lane's on.
template <bool WAVE>
__device__ __forceinline__ TileView tile_view(const TileArgs& t, const u32 gt) {
    constexpr int TH = kTileH, TW = kTileW;
    const u32 span = t.tile_end - t.tile_begin;
    TileView v;
    v.active = gt < span * (u32)t.B;
    const u32 tt = t.tile_begin + (v.active ? gt / (u32)t.B : 0u);
    const int b = v.active ? (int)(gt % (u32)t.B) : 0;
    u32 first;
    int o = slot_of(t.tile_start, t.NL, WAVE ? tt : (u32)uniform((int)tt), &first);
    if constexpr (!WAVE) o = slot_after(t.tile_start, t.NL, tt, o, &first);
    // (as region_tables_kernel lists the slots: a division instead of a load)
    const int r = (o % t.N) * t.L + (t.L - 1 - o / t.N);
    v.H = t.shapes[2 * r];
    v.W = t.shapes[2 * r + 1];
    v.start = t.starts[r];
    const u32 lt = tt - first;
    const u32 tpr = (u32)(v.W + TW - 1) / TW;
    v.ty = (int)(lt / tpr) * TH;
    v.tx = (int)(lt % tpr) * TW;
    v.cbase = (u32)b * t.cells_per_item + t.cell_start[r];
    v.row_base = (size_t)b * (size_t)t.R;
    v.vals = t.vals;
    v.off = t.off;
    v.frac = t.frac;
    v.w = t.w;
    v.w16 = (t.G & 3) == 0 && ((uintptr_t)t.w & 15) == 0;
    v.grad_out = t.grad_out;
    v.grad_feat = t.grad_feat;
    v.nrec = t.nrec;
    v.sample_offset = 0;
    v.sample_count = t.nrec;
    v.C = t.C;
    v.G = t.G;
    v.magic = t.magic;
    v.magic_shift = t.magic_shift;
    v.vscale = t.view_scale;
    v.N = t.N;
    v.L = t.L;
    return v;
}

// The same of a batch: tiles of all scenes' regions in slot order.
template <bool WAVE>
__device__ __forceinline__ TileView tile_view(const BatchArgs& b, const u32 gt) {
    constexpr int TH = kTileH, TW = kTileW;
    TileView v;
    v.active = gt < b.tile_end - b.tile_begin;
    const u32 tt = b.tile_begin + (v.active ? gt : 0u);
    u32 first;
    int slot = slot_of(b.t.tile_start, (int)b.total_regions, WAVE ? tt : (u32)uniform((int)tt),
                       &first);
    if constexpr (!WAVE) slot = slot_after(b.t.tile_start, (int)b.total_regions, tt, slot, &first);
    const int s = (int)b.t.slot_scene[slot];
    const int r = (int)b.t.slot_region[slot];
    const msda_scene& sc = b.scenes[s];
    v.H = sc.spatial_shapes[2 * r];
    v.W = sc.spatial_shapes[2 * r + 1];
    v.start = sc.level_start_index[r];
    const u32 lt = tt - first;
    const u32 tpr = (u32)(v.W + TW - 1) / TW;
    v.ty = (int)(lt / tpr) * TH;
    v.tx = (int)(lt % tpr) * TW;
    v.cbase = b.t.cell_start[b.t.region_start[s] + (u32)r];
    v.row_base = 0;
    v.vals = b.vals;
    v.off = b.off;
    v.frac = b.rec_frac;
    v.w = b.w32 ? b.w32 + (size_t)b.t.sample_start[s] * (size_t)b.G : sc.weights;
    v.w16 = (b.G & 3) == 0 && ((uintptr_t)v.w & 15) == 0;
    v.grad_out = sc.grad_out;
    v.grad_feat = sc.grad_feat;
    v.nrec = b.total_samples;
    v.sample_offset = b.t.sample_start[s];
    v.sample_count = b.t.sample_start[s + 1] - b.t.sample_start[s];
    v.C = b.C;
    v.G = b.G;
    v.magic = b.t.magic[s];
    v.magic_shift = (int)b.t.magic_shift[s];
    v.vscale = nullptr;
    v.N = 1;
    v.L = 1;
    return v;
}

// The tile of id gt by `waves` waves of the block, this wave the wt-th of them.
template <class OT, int CPL, bool WHOLE, int QB, class Args>
__device__ __forceinline__ void tile_body(const Args& t, const u32 gt, const int waves,
                                          const int wt) {
    static_assert(kTileH == 4 && kTileW == 4, "the cell dispatch is written for 4x4 tiles");
    // LDS: per wave a record table (64 entries of bilinear factors, anchor and G
    // weights); after the records, the waves' partial sums in its space
    extern __shared__ __align__(16) unsigned char smem[];
    tile_reduce<OT, CPL, WHOLE, QB>(tile_view<true>(t, gt), t.lps_shift, waves, wt,
                                    reinterpret_cast<float*>(smem));
}

// Sparse tiles from id gt on, one per sub-wave, t.sparse of them.
template <class OT, int CPL, class Args>
__device__ __forceinline__ void sparse_body(const Args& t, const u32 gt, u32 end, const int wave) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int sub = (threadIdx.x & 63) >> t.lps_shift;
    TileView v = tile_view<false>(t, min(gt + (u32)sub, end));
    v.active = v.active && sub < t.sparse;
    float* tab =
        reinterpret_cast<float*>(smem) + (size_t)wave * sparse_wave_floats(t.lps_shift, t.G);
    tile_reduce_sparse<OT, CPL>(v, t.lps_shift,
                                reinterpret_cast<u32*>(tab + 64 * tile_entry_floats(t.G)), tab);
}

// At most 128 VGPRs, i.e. 4 waves per SIMD. The reduction waits on record
// and grad_out loads, and a fourth wave hides more of that than a few more
// registers give (measured on the 64-camera scene: light tiles 0.28 -> 0.24
// ms, coarse 0.19 -> 0.18 ms).
//
// A light tile has about one record per cell, so its wave issues the first
// record's row of a cell row's five cells together (FIRST) and the rest two
// at a time; a coarse tile's wave has runs long enough for four at a time
// (64 cameras BF16 0.358 -> 0.345 ms, 6 cameras FP32 75 -> 67 us; 6 or 8 at a
// time 69 and 71, two and FIRST 79). Boundaries and anchors are lanes'
// registers, read as scalars: an LDS round trip per record less.
//
// Narrower records (C < 64 * CPL) share the wave as sub-waves of one tile
// rather than taking tiles of their own, which left a run-time dispatch on
// the cell per record and, on small problems, too few waves: 2 cameras of
// 128 x 224, C = 64, 128 anchors 144 -> 30 us, 32 cameras of 256 x 448, 900
// anchors, C = 128 285 -> 165 us, C = 64 317 -> 150 us. Sparse light tiles do
// take a sub-wave each (SPARSE, see sparse_tiles).
//
// One launch for both kinds of tiles: the coarse tiles (ids below
// (tile_split - tile_begin) * B) first, all waves of a block each, then the
// light ones, one wave each; the light blocks fill the CUs around the long
// coarse ones instead of waiting for them to drain. A block has 4 waves, or 8
// where the coarse tiles would be the launch's critical path (wide_tiles).
constexpr int kMaxTileBlockWaves = 8;

template <class OT, int CPL, bool WHOLE, bool SPARSE, int QB, class Args>
__device__ __forceinline__ void tile_block(const Args& t, const u32 items) {
    const int BW = (int)(blockDim.x >> 6);
    const u32 heavy = (t.tile_split - t.tile_begin) * items;
    const int wave = uniform((int)(threadIdx.x >> 6));
    if (blockIdx.x < heavy) {
        tile_body<OT, CPL, WHOLE, QB>(t, blockIdx.x, BW, wave);
        return;
    }
    const u32 w = (blockIdx.x - heavy) * (u32)BW + (u32)wave;
    if constexpr (SPARSE)
        sparse_body<OT, CPL>(t, heavy + w * (u32)t.sparse, (t.tile_end - t.tile_begin) * items,
                             wave);
    else
        tile_body<OT, CPL, WHOLE, 2>(t, heavy + w, 1, 0);
}

template <class OT, int CPL, bool WHOLE, bool SPARSE>
__global__ void __launch_bounds__(64 * kMaxTileBlockWaves)
    __attribute__((amdgpu_waves_per_eu(4, 8))) gfeat_tile_kernel(TileArgs t) {
    tile_block<OT, CPL, WHOLE, SPARSE, WHOLE ? 4 : 2>(t, (u32)t.B);
}

// The batched form; its heavy tiles ([tile_begin, tile_split)) too walk as the
// light ones do: with the batch's scene lookups, 4 rows at a time spilled under
// the 128-VGPR cap (the 12-scene batch's step: 9.37 ms with 4, 9.22 ms with 2).
template <class OT, int CPL, bool WHOLE, bool SPARSE>
__global__ void __launch_bounds__(64 * kMaxTileBlockWaves)
    __attribute__((amdgpu_waves_per_eu(4, 8))) gfeat_tile_batched_kernel(BatchArgs b) {
    tile_block<OT, CPL, WHOLE, SPARSE, 2>(b, 1);
}

// ---------------------------------------------------------------- launchers

// LDS of a tile block of `waves` waves: the larger of the record tables (sparse
// tiles: with the cell boundaries) and the partial sums (coarse tiles: waves/2
// halves of a tile's accumulators).
template <int CPL>
static size_t tile_lds_bytes(int waves, int G, bool coarse, int sparse, int lps_shift) {
    const size_t part = coarse ? (size_t)(waves / 2) * kTileH * kTileW * CPL * 64 * 4 : 0;
    const size_t wave = sparse ? sparse_wave_floats(lps_shift, G) : 64 * tile_entry_floats(G);
    const size_t tables = (size_t)waves * wave * sizeof(float);
    return part > tables ? part : tables;
}

// [tile_begin, tile_end), coarse up to tile_split: one launch, or as many as
// hold the waves (a tile of each of `items` batch items takes up to block_waves).
template <class Args, class F>
static hipError_t tile_parts(Args t, u32 items, F&& launch) {
    const u32 BW = (u32)t.block_waves, begin = t.tile_begin, split = t.tile_split, end = t.tile_end;
    const u32 most = (u32)(kMaxLaunchWaves / BW / items ? kMaxLaunchWaves / BW / items : 1);
    for (u32 at = begin; at < end; at = t.tile_end) {
        t.tile_begin = at;
        t.tile_end = end - at < most ? end : at + most;
        t.tile_split = split < at ? at : split < t.tile_end ? split : t.tile_end;
        const u32 heavy = (t.tile_split - t.tile_begin) * items;
        const u32 light = (t.tile_end - t.tile_split) * items;
        const u32 per_block = BW * (u32)(t.sparse ? t.sparse : 1);
        launch(t, heavy, heavy + (light + per_block - 1) / per_block);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <class OT, int CPL, bool WHOLE, bool SPARSE>
static hipError_t tile_launch_of(const TileArgs& a, hipStream_t s) {
    return tile_parts(a, (u32)a.B, [&](const TileArgs& t, u32 heavy, u32 blocks) {
        mark_begin("gfeat_tile_kernel", s);
        hipLaunchKernelGGL((gfeat_tile_kernel<OT, CPL, WHOLE, SPARSE>), dim3(blocks),
                           dim3(64 * t.block_waves),
                           tile_lds_bytes<CPL>(t.block_waves, t.G, heavy > 0, t.sparse, t.lps_shift),
                           s, t);
        mark_end(s);
    });
}

template <class OT, int CPL>
static hipError_t tile_launch(const TileArgs& t, hipStream_t s) {
    return t.lps_shift == 6 ? tile_launch_of<OT, CPL, true, false>(t, s)
           : t.sparse       ? tile_launch_of<OT, CPL, false, true>(t, s)
                            : tile_launch_of<OT, CPL, false, false>(t, s);
}

template <class OT, int CPL, bool WHOLE, bool SPARSE>
static hipError_t tile_batched_launch_of(const BatchArgs& a, hipStream_t s) {
    return tile_parts(a, 1, [&](const BatchArgs& b, u32 heavy, u32 blocks) {
        mark_begin("gfeat_tile_batched", s);
        hipLaunchKernelGGL((gfeat_tile_batched_kernel<OT, CPL, WHOLE, SPARSE>), dim3(blocks),
                           dim3(64 * b.block_waves),
                           tile_lds_bytes<CPL>(b.block_waves, b.G, heavy > 0, b.sparse, b.lps_shift),
                           s, b);
        mark_end(s);
    });
}

template <class OT, int CPL>
static hipError_t tile_batched_launch(const BatchArgs& b, hipStream_t s) {
    return b.lps_shift == 6 ? tile_batched_launch_of<OT, CPL, true, false>(b, s)
           : b.sparse       ? tile_batched_launch_of<OT, CPL, false, true>(b, s)
                            : tile_batched_launch_of<OT, CPL, false, false>(b, s);
}

hipError_t launch_gfeat_tiles_batched(const BatchArgs& b, int out_dtype, int cpl, hipStream_t s) {
    switch (out_dtype * 100 + cpl) {
        case kF32 * 100 + 1: return tile_batched_launch<TF32, 1>(b, s);
        case kF32 * 100 + 2: return tile_batched_launch<TF32, 2>(b, s);
        case kF32 * 100 + 4: return tile_batched_launch<TF32, 4>(b, s);
        case kBF16 * 100 + 1: return tile_batched_launch<TBF16, 1>(b, s);
        case kF16 * 100 + 1: return tile_batched_launch<TF16, 1>(b, s);
        case kBF16 * 100 + 2: return tile_batched_launch<TBF16, 2>(b, s);
        case kF16 * 100 + 2: return tile_batched_launch<TF16, 2>(b, s);
        case kBF16 * 100 + 4: return tile_batched_launch<TBF16, 4>(b, s);
        case kF16 * 100 + 4: return tile_batched_launch<TF16, 4>(b, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gfeat_tiles(const TileArgs& t, int out_dtype, int cpl, hipStream_t s) {
    switch (out_dtype * 100 + cpl) {
        case kF32 * 100 + 1: return tile_launch<TF32, 1>(t, s);
        case kF32 * 100 + 2: return tile_launch<TF32, 2>(t, s);
        case kF32 * 100 + 4: return tile_launch<TF32, 4>(t, s);
        case kBF16 * 100 + 1: return tile_launch<TBF16, 1>(t, s);
        case kF16 * 100 + 1: return tile_launch<TF16, 1>(t, s);
        case kBF16 * 100 + 2: return tile_launch<TBF16, 2>(t, s);
        case kF16 * 100 + 2: return tile_launch<TF16, 2>(t, s);
        case kBF16 * 100 + 4: return tile_launch<TBF16, 4>(t, s);
        case kF16 * 100 + 4: return tile_launch<TF16, 4>(t, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_region_tables(const int32_t* shapes, int32_t N, int32_t L, u32* cell_start,
                                u32* tile_start, hipStream_t s) {
    mark_begin("region_tables", s);
    hipLaunchKernelGGL(region_tables_kernel, dim3(1), dim3(256), 0, s, shapes, N, L, cell_start,
                       tile_start);
    mark_end(s);
    return hipGetLastError();
}

}  // namespace msda
