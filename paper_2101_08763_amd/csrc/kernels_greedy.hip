// kernels_greedy.hip -- the small kernels of the on-device Greedy optimizer
// (Algorithm 1): state initialisation and the deterministic argmax that picks
// each round's element without a round trip to the host.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "internal.h"

namespace exemcl {

namespace {

constexpr int kThreads = 256;
constexpr int64_t kMaxBlocks = 1024;
constexpr int64_t kItemsPerBlock = 16 * kThreads;

// (v, i) beats (bv, bi) when larger, or equal with a lower index: the
// lowest candidate position wins ties.
__device__ inline void take(float &bv, int32_t &bi, float v, int32_t i) {
    if (v > bv || (v == bv && i < bi)) {
        bv = v;
        bi = i;
    }
}

// Block-wide best pair; the result is valid in thread 0.
__device__ inline void block_best(float &bv, int32_t &bi) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        const float ov = __shfl_xor(bv, off);
        const int32_t oi = __shfl_xor(bi, off);
        take(bv, bi, ov, oi);
    }
    __shared__ float sv[kThreads / 64];
    __shared__ int32_t si[kThreads / 64];
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sv[w] = bv;
        si[w] = bi;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int q = 1; q < kThreads / 64; ++q) take(bv, bi, sv[q], si[q]);
}

__global__ __launch_bounds__(kThreads) void greedy_init_kernel(int32_t *__restrict__ cands,
                                                               uint8_t *__restrict__ taken,
                                                               float *__restrict__ g, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    cands[i] = (int32_t)i;
    taken[i] = 0;
    g[i] = 0.0f;  // S empty: only e0, whose h is 0 everywhere
}

// Stage 1: the best untaken candidate of each block's grid-stride share.  A
// NaN score ranks below every number.
__global__ __launch_bounds__(kThreads) void argmax_blocks_kernel(const float *__restrict__ scores,
                                                                 const uint8_t *__restrict__ taken, int64_t n,
                                                                 float *__restrict__ pval,
                                                                 int32_t *__restrict__ pidx) {
    float bv = -INFINITY;
    int32_t bi = INT32_MAX;
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += stride) {
        if (taken[i]) continue;
        float v = scores[i];
        if (isnan(v)) v = -INFINITY;
        take(bv, bi, v, (int32_t)i);
    }
    block_best(bv, bi);
    if (threadIdx.x == 0) {
        pval[blockIdx.x] = bv;
        pidx[blockIdx.x] = bi;
    }
}

// Stage 2 (one block): the overall best; record it as this round's element,
// its score as f of the grown set, and mark it taken.
__global__ __launch_bounds__(kThreads) void argmax_final_kernel(const float *__restrict__ pval,
                                                                const int32_t *__restrict__ pidx, int64_t nb,
                                                                const float *__restrict__ scores,
                                                                uint8_t *__restrict__ taken, int64_t n,
                                                                int32_t *__restrict__ S_slot,
                                                                float *__restrict__ f_slot) {
    float bv = -INFINITY;
    int32_t bi = INT32_MAX;
    for (int64_t b = threadIdx.x; b < nb; b += kThreads) take(bv, bi, pval[b], pidx[b]);
    block_best(bv, bi);
    if (threadIdx.x == 0) {
        if (bi >= 0 && bi < n) {
            *S_slot = bi;
            *f_slot = scores[bi];
            taken[bi] = 1;
        } else {  // nothing left to take (the host never asks for that)
            *S_slot = kEmptySlot;
            *f_slot = __builtin_nanf("");
        }
    }
}

// ---------------------------------------------------------------------------
// Lazy rounds (see internal.h).  The filter combines four rounded scores --
// the candidate's in an earlier round, f then, f now, the best score now --
// and stands for a fifth, the candidate's now.  Their h_s(v) have the same
// bits in every round, kernel and launch shape (one order of the same
// instructions: scoring and cache must keep it), and of fixed numbers the sum
// of maxima is exactly submodular, so only the rounding of the sums counts.
// All terms are >= 0 and a score passes 8 roundings: 6 fp32 additions in a
// wavefront, its workgroup's sum, the result.  Scores are at most L({e0}), so
// five of them and the three operations in between stay below
// (5 * 8 + 3) 2^-24 L({e0}) < 64 * 2^-24 L({e0}), for any data.  The filter's
// tol, (16 sqrt(d) + 64) 2^-24 L({e0}), leaves four times that at d = 100.
// ---------------------------------------------------------------------------
constexpr int kPickThreads = 1024;

__global__ __launch_bounds__(kPickThreads) void greedy_scale_kernel(const float *__restrict__ q, int64_t n, double c,
                                                                    GreedyState *__restrict__ state) {
    __shared__ double part[kPickThreads];
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += kPickThreads) s += (double)q[i];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int w = kPickThreads / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        state->tol = (float)(c * part[0] / (double)n);
        state->count = 0;
    }
}

__global__ __launch_bounds__(kThreads) void greedy_probe_kernel(const float *__restrict__ estimate,
                                                                const uint8_t *__restrict__ taken, int64_t n,
                                                                int32_t *__restrict__ probes) {
    const int64_t lo = blockIdx.x * n / kGreedyProbes, hi = (blockIdx.x + 1) * n / kGreedyProbes;
    float bv = -INFINITY;
    int32_t bi = INT32_MAX;
    for (int64_t i = lo + threadIdx.x; i < hi; i += kThreads) {
        if (taken[i]) continue;
        const float v = estimate[i];
        take(bv, bi, isnan(v) ? -INFINITY : v, (int32_t)i);
    }
    block_best(bv, bi);
    if (threadIdx.x == 0) probes[blockIdx.x] = bi < n ? bi : kEmptySlot;
}

__global__ __launch_bounds__(kThreads) void greedy_filter_kernel(const float *__restrict__ gain,
                                                                 const uint8_t *__restrict__ taken, int64_t n,
                                                                 const int32_t *__restrict__ probes,
                                                                 const float *__restrict__ probe_scores,
                                                                 const float *__restrict__ f_prev,
                                                                 GreedyState *__restrict__ state,
                                                                 int32_t *__restrict__ list) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    float best = -INFINITY;
    bool probed = false;
    for (int b = 0; b < kGreedyProbes; ++b) {  // uniform addresses
        const int32_t c = probes[b];
        if (c >= 0) best = fmaxf(best, probe_scores[b]);
        probed |= c == i;
    }
    // a NaN anywhere keeps the candidate
    const bool keep = i < n && !probed && !taken[i] && !(gain[i] + *f_prev < best - state->tol);
    const uint64_t mask = __ballot(keep);
    if (mask == 0) return;
    const int lane = threadIdx.x & 63, first = __ffsll((unsigned long long)mask) - 1;
    int at = 0;
    if (lane == first) at = atomicAdd(&state->count, __popcll(mask));
    at = __shfl(at, first);
    if (keep) list[at + __popcll(mask & ((1ull << lane) - 1))] = (int32_t)i;
}

__global__ __launch_bounds__(kPickThreads) void greedy_pick_kernel(
    const int32_t *__restrict__ probes, const float *__restrict__ probe_scores, const int32_t *__restrict__ list,
    const float *__restrict__ list_scores, const float *__restrict__ f_prev, GreedyState *__restrict__ state,
    float *__restrict__ gain, uint8_t *__restrict__ taken, int64_t n, int32_t *__restrict__ S_slot,
    float *__restrict__ f_slot) {
    __shared__ float sv[kPickThreads];
    __shared__ int32_t si[kPickThreads];
    const int count = state->count, tid = threadIdx.x;
    const float f = *f_prev;
    float bv = -INFINITY, braw = 0.0f;
    int32_t bi = INT32_MAX;
    for (int j = tid - kGreedyProbes; j < count; j += kPickThreads) {
        const int32_t c = j < 0 ? probes[j + kGreedyProbes] : list[j];
        if (c < 0) continue;
        const float s = j < 0 ? probe_scores[j + kGreedyProbes] : list_scores[j];
        gain[c] = s - f;
        take(bv, bi, isnan(s) ? -INFINITY : s, c);
        if (bi == c) braw = s;
    }
    sv[tid] = bv;
    si[tid] = bi;
    __syncthreads();
    for (int w = kPickThreads / 2; w >= 1; w >>= 1) {
        if (tid < w) take(sv[tid], si[tid], sv[tid + w], si[tid + w]);
        __syncthreads();
    }
    if (bi == si[0] && bi < n) {  // the one thread that scored it
        *S_slot = bi;
        *f_slot = braw;
        taken[bi] = 1;
    }
    if (tid == 0) {
        state->count = 0;
        if (si[0] >= n) {  // nothing left to take (the host never asks for that)
            *S_slot = kEmptySlot;
            *f_slot = __builtin_nanf("");
        }
    }
}

}  // namespace

hipError_t launch_greedy_scale(const float *q, int64_t n, int64_t d, GreedyState *state, hipStream_t st) {
    const double c = (16.0 * sqrt((double)d) + 64.0) * 0x1p-24;
    hipLaunchKernelGGL(greedy_scale_kernel, dim3(1), dim3(kPickThreads), 0, st, q, n, c, state);
    return hipGetLastError();
}

hipError_t launch_greedy_probe(const float *estimate, const uint8_t *taken, int64_t n, int32_t *probes, hipStream_t st) {
    hipLaunchKernelGGL(greedy_probe_kernel, dim3(kGreedyProbes), dim3(kThreads), 0, st, estimate, taken, n, probes);
    return hipGetLastError();
}

hipError_t launch_greedy_filter(const float *gain, const uint8_t *taken, int64_t n, const int32_t *probes,
                                const float *probe_scores, const float *f_prev, GreedyState *state, int32_t *list,
                                hipStream_t st) {
    hipLaunchKernelGGL(greedy_filter_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                       gain, taken, n, probes, probe_scores, f_prev, state, list);
    return hipGetLastError();
}

hipError_t launch_greedy_pick(const int32_t *probes, const float *probe_scores, const int32_t *list,
                              const float *list_scores, const float *f_prev, GreedyState *state, float *gain,
                              uint8_t *taken, int64_t n, int32_t *S_slot, float *f_slot, hipStream_t st) {
    hipLaunchKernelGGL(greedy_pick_kernel, dim3(1), dim3(kPickThreads), 0, st, probes, probe_scores, list, list_scores,
                       f_prev, state, gain, taken, n, S_slot, f_slot);
    return hipGetLastError();
}

int64_t argmax_blocks(int64_t n) {
    int64_t b = (n + kItemsPerBlock - 1) / kItemsPerBlock;
    return b < 1 ? 1 : (b > kMaxBlocks ? kMaxBlocks : b);
}

hipError_t launch_greedy_init(int32_t *cands, uint8_t *taken, float *g, int64_t n, hipStream_t st) {
    hipLaunchKernelGGL(greedy_init_kernel, dim3((unsigned)((n + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                       cands, taken, g, n);
    return hipGetLastError();
}

hipError_t launch_argmax(const float *scores, uint8_t *taken, int64_t n, float *pval, int32_t *pidx,
                         int32_t *S_slot, float *f_slot, hipStream_t st) {
    const int64_t nb = argmax_blocks(n);
    hipLaunchKernelGGL(argmax_blocks_kernel, dim3((unsigned)nb), dim3(kThreads), 0, st, scores, taken, n, pval, pidx);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(argmax_final_kernel, dim3(1), dim3(kThreads), 0, st, pval, pidx, nb, scores, taken, n, S_slot,
                       f_slot);
    return hipGetLastError();
}

}  // namespace exemcl
