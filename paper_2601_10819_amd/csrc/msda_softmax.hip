// Fused weight generation: the per-group softmax that turns the weight
// logits into MSDA's weights (over the P*N*L (keypoint, camera, level)
// entries of each (batch item, anchor, group)), and its gradient.
//
// The forward never writes the weights: softmax_kernel reduces each group's
// logits to (max, 1/sum of exp) and the gathers apply exp(logit - max) / sum
// while they stage the weights. The backward has the same kernel write the
// FP32 weights once, runs the plain backward on them, and
// softmax_grad_kernel maps grad_weights to the logits' gradient in place:
// d logit = w * (d w - sum over the group of w * d w).
//
// Each pass is bound by its bytes and by how many of them are in flight, so
// one workgroup takes an anchor's n = P*N*L*G entries (groups fastest) from
// the first read to the last write: nothing but the result goes to memory,
// no launch merges partials, and a second look at the entries finds them in
// registers (the last kRound per thread) or near. A thread's kRound loads of
// a round are unconditional -- past the end, the last entry, whose value is
// then replaced -- so that all are in flight together; behind a branch each,
// the compiler waits for one before it issues the next. 900 anchors of 64
// cameras, 13 keypoints, 4 levels and 8 groups (96 MB of FP32 logits):
// statistics 41 -> 26 us (3.7 TB/s), weights for the backward 77 -> 51 (3.8
// TB/s), the gradient 77 -> 79 in one launch instead of three.
//
// G is a power of two <= 64, so entry e of an anchor belongs to group e % G
// and thread t sees only group t % G; the threads of a group are combined in
// a fixed order (bitwise reproducible).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "msda_common.h"

namespace msda {

namespace {

constexpr int kRound = 16;            // entries per thread and round
constexpr int kFlatThreads = 256;
constexpr size_t kFlatChunk = (size_t)kRound * kFlatThreads;

__device__ __forceinline__ float widen(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }
__device__ __forceinline__ float widen(float v) { return v; }

// Entries t, t + THREADS, ... (kRound of them) of p[0, left), left > 0; the
// last entry instead of those past the end.
template <int THREADS, class T>
__device__ __forceinline__ void load_round(const T* p, size_t left, float* x) {
    const uint32_t t = threadIdx.x;
    T raw[kRound];
    if (left >= (size_t)kRound * THREADS) {
#pragma unroll
        for (int k = 0; k < kRound; ++k) raw[k] = p[t + (uint32_t)(k * THREADS)];
    } else {
        const uint32_t end = (uint32_t)left - 1;
#pragma unroll
        for (int k = 0; k < kRound; ++k) raw[k] = p[min(t + (uint32_t)(k * THREADS), end)];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < kRound; ++k) x[k] = widen(raw[k]);
}

// Whether entry t + k * THREADS of a round is one of the `left` that are left.
template <int THREADS>
__device__ __forceinline__ bool in_round(int k, size_t left) {
    return left >= (size_t)kRound * THREADS || threadIdx.x + (uint32_t)(k * THREADS) < (uint32_t)left;
}

// (max, sum of exp(x - max)) of two disjoint sets.
__device__ __forceinline__ float2 merge(float2 a, float2 b) {
    if (b.y == 0.f) return a;
    if (a.y == 0.f) return b;
    const float m = fmaxf(a.x, b.x);
    return make_float2(m, a.y * expf(a.x - m) + b.y * expf(b.x - m));
}

// The combined value of the threads that share a group (t % G), in each of
// them: within the wave by xor steps over the lane bits above log2(G), then
// the waves in order through LDS.
template <int THREADS, class F>
__device__ __forceinline__ float group_total(float v, int G, float* lds, F combine) {
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = t & (G - 1);
    for (int m = G; m < 64; m <<= 1) v = combine(v, __shfl_xor(v, m, 64));
    if (lane < G) lds[wave * 64 + lane] = v;
    __syncthreads();
    v = lds[g];
    for (int w = 1; w < THREADS / 64; ++w) v = combine(v, lds[w * 64 + g]);
    __syncthreads();
    return v;
}

// (max, sum of exp(x - max)) of a thread's entries of a round with `left` left.
template <int THREADS>
__device__ __forceinline__ float2 round_stats(float* x, size_t left) {
    float m = -INFINITY;
#pragma unroll
    for (int k = 0; k < kRound; ++k) {
        if (!in_round<THREADS>(k, left)) x[k] = -INFINITY;
        m = fmaxf(m, x[k]);
    }
    float sum = 0.f;
    // exp(-inf) = 0; only masked entries: nothing to add, but a NaN stays one
#pragma unroll
    for (int k = 0; k < kRound; ++k)
        sum += m != -INFINITY ? expf(x[k] - m) : (x[k] == x[k] ? 0.f : x[k]);
    return make_float2(m, sum);
}

// A block's (max, sum of exp) per group, in each of the group's threads.
template <int THREADS>
__device__ __forceinline__ float2 group_stats(float2 acc, int G, float* lds) {
    const float m = group_total<THREADS>(acc.x, G, lds, [](float a, float b) { return fmaxf(a, b); });
    const float mine = acc.y == 0.f ? 0.f : acc.y * expf(acc.x - m);
    return make_float2(m, group_total<THREADS>(mine, G, lds, [](float a, float b) { return a + b; }));
}

// One anchor per block: the groups' (max, 1/sum of exp) to `stats` and the
// weights to `weights`, either of which may be nullptr.
template <class T, int THREADS>
__global__ void __launch_bounds__(THREADS) softmax_kernel(const T* logits, size_t n, int G,
                                                          float2* stats, float* weights) {
    __shared__ float lds[THREADS];
    const size_t ba = blockIdx.x, t = threadIdx.x;
    const T* p = logits + ba * n;
    constexpr size_t kStep = (size_t)kRound * THREADS;
    const size_t last = (n - 1) / kStep * kStep;      // the last round's first entry
    float x[kRound];
    float2 acc = make_float2(-INFINITY, 0.f);
    for (size_t r = 0;; r += kStep) {
        load_round<THREADS>(p + r, n - r, x);
        acc = merge(acc, round_stats<THREADS>(x, n - r));
        if (r == last) break;
    }
    const float2 all = group_stats<THREADS>(acc, G, lds);
    const float m = all.x, inv = 1.f / all.y;
    if (stats && t < (size_t)G) stats[ba * G + t] = make_float2(m, inv);
    if (!weights) return;
    float* w = weights + ba * n;
    for (size_t r = last;; r -= kStep) {              // x holds the last round's logits
#pragma unroll
        for (int k = 0; k < kRound; ++k) {
            const float v = expf(x[k] - m) * inv;
            if (in_round<THREADS>(k, n - r)) w[r + t + (uint32_t)(k * THREADS)] = v;
        }
        if (r == 0) break;
        load_round<THREADS>(p + r - kStep, kStep, x);
    }
}

// BF16 weights widened to FP32, all `n` of them.
__global__ void __launch_bounds__(kFlatThreads) weights_f32_kernel(const uint16_t* src, size_t n,
                                                                    float* w) {
    const size_t e0 = (size_t)blockIdx.x * kFlatChunk + threadIdx.x;
    float x[kRound];
    load_round<kFlatThreads>(src + (size_t)blockIdx.x * kFlatChunk,
                              n - (size_t)blockIdx.x * kFlatChunk, x);
#pragma unroll
    for (int k = 0; k < kRound; ++k) {
        const size_t e = e0 + (size_t)k * kFlatThreads;
        if (e < n) w[e] = x[k];
    }
}

// One anchor per block: grad = w * (grad - D), D the group's sum of w * grad.
template <int THREADS>
__global__ void __launch_bounds__(THREADS) softmax_grad_kernel(const float* weights, float* grads,
                                                               size_t n, int G) {
    __shared__ float lds[THREADS];
    const size_t ba = blockIdx.x, t = threadIdx.x;
    const float* w = weights + ba * n;
    float* grad = grads + ba * n;
    constexpr size_t kStep = (size_t)kRound * THREADS;
    const size_t last = (n - 1) / kStep * kStep;
    float x[kRound], y[kRound];
    float acc = 0.f;
    for (size_t r = 0;; r += kStep) {
        load_round<THREADS>(w + r, n - r, x);
        load_round<THREADS>(grad + r, n - r, y);
#pragma unroll
        for (int k = 0; k < kRound; ++k)
            if (in_round<THREADS>(k, n - r)) acc = fmaf(x[k], y[k], acc);
        if (r == last) break;
    }
    const float d = group_total<THREADS>(acc, G, lds, [](float a, float b) { return a + b; });
    for (size_t r = last;; r -= kStep) {              // x, y hold the last round
#pragma unroll
        for (int k = 0; k < kRound; ++k) {
            if (in_round<THREADS>(k, n - r))
                grad[r + t + (uint32_t)(k * THREADS)] = x[k] * (y[k] - d);
        }
        if (r == 0) break;
        load_round<THREADS>(w + r - kStep, kStep, x);
        load_round<THREADS>(grad + r - kStep, kStep, y);
    }
}

// Few anchors of many entries: an anchor's entries in `parts` runs of `per`, a
// block each (blockIdx.x), whose partial results go through `part`, [anchor][run]
// [group], to a second launch.
template <class T>
__global__ void __launch_bounds__(kFlatThreads) softmax_part_kernel(const T* logits, size_t n, int G,
                                                                    size_t per, float2* part) {
    __shared__ float lds[kFlatThreads];
    const size_t ba = blockIdx.y, lo = blockIdx.x * per, hi = min(lo + per, n);
    float x[kRound];
    float2 acc = make_float2(-INFINITY, 0.f);
    for (size_t r = lo; r < hi; r += kFlatChunk) {
        load_round<kFlatThreads>(logits + ba * n + r, hi - r, x);
        acc = merge(acc, round_stats<kFlatThreads>(x, hi - r));
    }
    acc = group_stats<kFlatThreads>(acc, G, lds);
    if (threadIdx.x < (unsigned)G) part[(ba * gridDim.x + blockIdx.x) * G + threadIdx.x] = acc;
}

template <class T>
__global__ void __launch_bounds__(kFlatThreads) softmax_weights_kernel(const T* logits, size_t n,
                                                                       int G, size_t per,
                                                                       const float2* part,
                                                                       float* weights) {
    const size_t ba = blockIdx.y, lo = blockIdx.x * per, hi = min(lo + per, n);
    const float2* mine = part + ba * gridDim.x * G + (threadIdx.x & (unsigned)(G - 1));
    float2 all = make_float2(-INFINITY, 0.f);
    for (unsigned k = 0; k < gridDim.x; ++k) all = merge(all, mine[(size_t)k * G]);
    const float inv = 1.f / all.y;
    float x[kRound];
    for (size_t r = lo; r < hi; r += kFlatChunk) {
        load_round<kFlatThreads>(logits + ba * n + r, hi - r, x);
#pragma unroll
        for (int k = 0; k < kRound; ++k)
            if (in_round<kFlatThreads>(k, hi - r))
                weights[ba * n + r + threadIdx.x + (uint32_t)(k * kFlatThreads)] =
                    expf(x[k] - all.x) * inv;
    }
}

__global__ void __launch_bounds__(kFlatThreads) softmax_dot_kernel(const float* weights,
                                                                   const float* grads, size_t n,
                                                                   int G, size_t per, float* part) {
    __shared__ float lds[kFlatThreads];
    const size_t ba = blockIdx.y, lo = blockIdx.x * per, hi = min(lo + per, n);
    float x[kRound], y[kRound], acc = 0.f;
    for (size_t r = lo; r < hi; r += kFlatChunk) {
        load_round<kFlatThreads>(weights + ba * n + r, hi - r, x);
        load_round<kFlatThreads>(grads + ba * n + r, hi - r, y);
#pragma unroll
        for (int k = 0; k < kRound; ++k)
            if (in_round<kFlatThreads>(k, hi - r)) acc = fmaf(x[k], y[k], acc);
    }
    acc = group_total<kFlatThreads>(acc, G, lds, [](float a, float b) { return a + b; });
    if (threadIdx.x < (unsigned)G) part[(ba * gridDim.x + blockIdx.x) * G + threadIdx.x] = acc;
}

__global__ void __launch_bounds__(kFlatThreads) softmax_apply_kernel(const float* weights,
                                                                     float* grads, size_t n, int G,
                                                                     size_t per,
                                                                     const float* part) {
    const size_t ba = blockIdx.y, lo = blockIdx.x * per, hi = min(lo + per, n);
    const float* mine = part + ba * gridDim.x * G + (threadIdx.x & (unsigned)(G - 1));
    float d = 0.f;
    for (unsigned k = 0; k < gridDim.x; ++k) d += mine[(size_t)k * G];
    float x[kRound], y[kRound];
    for (size_t r = lo; r < hi; r += kFlatChunk) {
        load_round<kFlatThreads>(weights + ba * n + r, hi - r, x);
        load_round<kFlatThreads>(grads + ba * n + r, hi - r, y);
#pragma unroll
        for (int k = 0; k < kRound; ++k)
            if (in_round<kFlatThreads>(k, hi - r))
                grads[ba * n + r + threadIdx.x + (uint32_t)(k * kFlatThreads)] = x[k] * (y[k] - d);
    }
}

// Runs an anchor is cut into, and their length: where a block per anchor leaves
// most of the 256 CUs without one and an anchor is many rounds long, as many as
// give every CU two blocks (64 cameras, 13 keypoints, 4 levels, 64 groups, 52
// rounds, whole gradient of the logits: 4 anchors 138 us in one block each, 82 in
// runs; 32 182 and 95; 100 359 and 247; 8 groups, 7 rounds, were no slower than
// two launches: 4 anchors 40 us).
struct Runs {
    unsigned parts;
    size_t per;
};

Runs runs_of(int64_t BA, size_t n) {
    const size_t rounds = (n + kFlatChunk - 1) / kFlatChunk;
    if (BA >= 128 || rounds < 8) return Runs{1, n};
    const size_t want = (size_t)(512 / BA);
    const size_t per = (rounds + want - 1) / want;
    return Runs{(unsigned)((rounds + per - 1) / per), per * kFlatChunk};
}

// Threads per anchor. Small anchors are one round of 256 threads. Otherwise
// 1024 threads read an anchor in few rounds where there are no more anchors
// than two per CU, and 512 where there are: 900 anchors of 26,624 entries are
// then all resident at once (statistics 26 us, with 1024 threads 34; weights
// 51 and 57). The gradient has two values per entry to read again if they are
// not one round, and 1024 threads hold more of them (79 us, with 512 85).
int threads_of(size_t n, int BA, bool gradient) {
    if (n <= kRound * 256) return 256;
    return BA <= 512 || (gradient && n > kRound * 512) ? 1024 : 512;
}

// f(int_c<threads>).
template <int I>
using int_c = std::integral_constant<int, I>;

template <class F>
void with_threads(int threads, F&& f) {
    if (threads == 256) f(int_c<256>{});
    else if (threads == 512) f(int_c<512>{});
    else f(int_c<1024>{});
}

// f(first anchor, anchors) over parts of fewer than 2^32 threads.
template <class F>
void in_parts(int BA, F&& f) {
    constexpr int kPart = 1 << 21;
    for (int64_t at = 0; at < BA; at += kPart)
        f((size_t)at, (unsigned)(BA - at < kPart ? BA - at : kPart));
}

template <class T>
void run_softmax(const void* logits, int BA, size_t n, int G, float2* stats, float* w,
                 hipStream_t s) {
    with_threads(threads_of(n, BA, false), [&](auto threads) {
        constexpr int THREADS = decltype(threads)::value;
        in_parts(BA, [&](size_t at, unsigned anchors) {
            hipLaunchKernelGGL((softmax_kernel<T, THREADS>), dim3(anchors), dim3(THREADS), 0, s,
                               static_cast<const T*>(logits) + at * n, n, G,
                               stats ? stats + at * (size_t)G : nullptr, w ? w + at * n : nullptr);
        });
    });
}

}  // namespace

size_t softmax_scratch_bytes(int64_t BA, size_t n, int G) {
    if (BA <= 0) return 0;
    const Runs runs = runs_of(BA, n);
    return runs.parts > 1 ? (size_t)BA * runs.parts * (size_t)G * sizeof(float2) : 0;
}

hipError_t launch_softmax(const void* logits, bool bf16, int BA, int PNL, int G, float2* stats,
                          float* weights, float2* scratch, hipStream_t s) {
    if (BA <= 0) return hipSuccess;
    const size_t n = (size_t)PNL * G;
    const Runs runs = runs_of(BA, n);
    if (!stats && scratch && runs.parts > 1) {
        const dim3 grid(runs.parts, (unsigned)BA);
        auto both = [&](auto* p) -> hipError_t {
            using T = std::remove_const_t<std::remove_pointer_t<decltype(p)>>;
            mark_begin("softmax_part", s);
            hipLaunchKernelGGL((softmax_part_kernel<T>), grid, dim3(kFlatThreads), 0, s, p, n, G,
                               runs.per, scratch);
            mark_end(s);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
            mark_begin("softmax", s);
            hipLaunchKernelGGL((softmax_weights_kernel<T>), grid, dim3(kFlatThreads), 0, s, p, n, G,
                               runs.per, scratch, weights);
            mark_end(s);
            return hipGetLastError();
        };
        return bf16 ? both(static_cast<const uint16_t*>(logits))
                    : both(static_cast<const float*>(logits));
    }
    mark_begin("softmax", s);
    if (bf16) run_softmax<uint16_t>(logits, BA, n, G, stats, weights, s);
    else run_softmax<float>(logits, BA, n, G, stats, weights, s);
    mark_end(s);
    return hipGetLastError();
}

hipError_t launch_weights_f32(const void* src, int BA, int PNL, int G, float* w, hipStream_t s) {
    if (BA <= 0) return hipSuccess;
    const size_t n = (size_t)BA * PNL * G;
    mark_begin("weights_f32", s);
    hipLaunchKernelGGL(weights_f32_kernel, dim3((unsigned)((n + kFlatChunk - 1) / kFlatChunk)),
                       dim3(kFlatThreads), 0, s, static_cast<const uint16_t*>(src), n, w);
    mark_end(s);
    return hipGetLastError();
}

hipError_t launch_softmax_grad(const float* w, float* grad, int BA, int PNL, int G, float2* scratch,
                               hipStream_t s) {
    if (BA <= 0) return hipSuccess;
    const size_t n = (size_t)PNL * G;
    const Runs runs = runs_of(BA, n);
    if (scratch && runs.parts > 1) {
        const dim3 grid(runs.parts, (unsigned)BA);
        float* part = reinterpret_cast<float*>(scratch);
        mark_begin("softmax_dot", s);
        hipLaunchKernelGGL(softmax_dot_kernel, grid, dim3(kFlatThreads), 0, s, w, grad, n, G,
                           runs.per, part);
        mark_end(s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        mark_begin("softmax_grad", s);
        hipLaunchKernelGGL(softmax_apply_kernel, grid, dim3(kFlatThreads), 0, s, w, grad, n, G,
                           runs.per, part);
        mark_end(s);
        return hipGetLastError();
    }
    mark_begin("softmax_grad", s);
    with_threads(threads_of(n, BA, true), [&](auto threads) {
        constexpr int THREADS = decltype(threads)::value;
        in_parts(BA, [&](size_t at, unsigned anchors) {
            hipLaunchKernelGGL((softmax_grad_kernel<THREADS>), dim3(anchors), dim3(THREADS), 0, s,
                               w + at * n, grad + at * n, n, G);
        });
    });
    mark_end(s);
    return hipGetLastError();
}

}  // namespace msda
