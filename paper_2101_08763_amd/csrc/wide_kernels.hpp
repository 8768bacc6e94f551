// wide_kernels.hpp -- evaluation of long fp16/bf16 rows as a tiled matrix
// product (instantiated in kernels_mfma_wide.hip).
//
// Above 1 024 coordinates a wavefront's registers do not hold its points.  The
// kernel in bigd_kernels.hpp keeps them by splitting the coordinates over the
// wavefronts, but a block of 32 points then reads every exemplar from L2 for
// itself, which bounds it at a quarter of the matrix cores' rate.  Here both
// operands go through LDS: a workgroup of 8 wavefronts computes 32 RT points
// x 256 exemplar columns at a time, 64 coordinates per stage, two stages in
// flight.  A wavefront holds RT x 4 accumulator tiles (RT row tiles of 16
// points, 4 column groups of 16 sets): RT + 4 fragments from LDS feed 4 RT
// instructions.  At 1.06 PFLOP/s the matrix cores are busy 55 % and LDS reads
// 21 % of the time; the rest are waits between stages.  20 000 x 1 536 bf16,
// 512 sets of 16: 1 040 us on the kernel in bigd_kernels.hpp, 477 here.
//
// Columns: 8 streams of staged tiles (16 sets, two members each; the layout
// of mfma_kernels.hpp), two per wavefront column.  PARTS = 1: a stream walks
// all tiles of its own set group; PARTS = 2: the two streams of a wavefront
// share a set group's tiles.  The maximum over a set's members does not
// depend on that choice, so the launch takes whichever balances better.
// Likewise RT: partial sums are written per 32 points, in the same order for
// every RT, so results do not depend on it.
#pragma once

#include <algorithm>
#include <atomic>

#include <hip/hip_ext.h>

#include "device.hpp"
#include "internal.h"
#include "mfma_kernels.hpp"

namespace exemcl {

constexpr int kWideWaves = 8, kWideStreams = 8;
constexpr int kWideRows = 32;                    // points per partial-sum row
constexpr int64_t kWideMaxD = int64_t(1) << 20;  // 256 rows within 32-bit byte offsets
constexpr int wide_stage(int rt) { return (2 * rt * 2 + kWideStreams * 4) * 1024; }

template <typename T, int RT, int PARTS>
__global__ __launch_bounds__(kWideWaves * 64, 2) void eval_wide_kernel(const T *__restrict__ V, int64_t n, int ld, int nkb,
                                                                       const unsigned char *__restrict__ tiles, int kt,
                                                                       int ngroups, int nrb, float *__restrict__ partials,
                                                                       int64_t lpad) {
    using M = Mfma<T, 16>;
    using vec_t = typename M::vec_t;
    constexpr int NB = 2, BM = 2 * RT * 16, SB = wide_stage(RT);
    constexpr int HDR = (16 * NB * 4 + 127) / 128 * 128;
    constexpr int GPB = kWideStreams / PARTS;  // set groups per column block
    constexpr int AF = RT / 2;                 // A fragments a wavefront stages (of 4 RT)
    static_assert(M::NB == NB && RT % 2 == 0 && 2 * SB <= kLdsBytes, "geometry");
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, grp = lane >> 4;
    const int wm = wave & 1, wn = wave >> 1;
    const int64_t tbytes = HDR + (int64_t)nkb * NB * 1024;
    const int rounds = (kt + PARTS - 1) / PARTS;
    const int ksteps = (nkb + 1) / 2;

    // Units (row block, column block).  Workgroups b, b + 8, b + 16, ... share
    // an XCD and its L2: they take consecutive units, up to 8 column blocks of
    // one row block side by side, so that each operand is fetched once for
    // several of them.
    const int ncb = (ngroups + GPB - 1) / GPB;
    const int units = nrb * ncb;
    const int per = (units + 7) / 8;
    const int b = (int)flat_block(), pos = b >> 3, u = (b & 7) * per + pos;
    if (pos >= per || u >= units) return;
    const int strip = u / (nrb * 8), width = min(8, ncb - strip * 8);
    const int in = u - strip * nrb * 8;
    const int rb = in / width, cb = strip * 8 + in % width;

    const int64_t row0 = (int64_t)rb * BM;
    const int64_t wrows = min((int64_t)BM, n - row0);
    const auto vwin = window_rsrc(V + row0 * (int64_t)ld, (uint32_t)(wrows * ld * (int64_t)sizeof(T)));

    // Stage st = (round, k-step) into buffer st % 2.  A fragments f = row
    // tile * 2 + k-block, this wavefront's AF * wave ...; then each stream's
    // four fragments (k-block, member).  What lies past the data reads as
    // zeros.
    int is_r = 0, is_k = 0;  // the stage to issue next
    auto issue = [&](int st) {
        unsigned char *buf = smem + (st & 1) * SB;
#pragma unroll
        for (int i = 0; i < AF; ++i) {
            const int f = wave * AF + i, kb = is_k * 2 + (f & 1), row = (f >> 1) * 16 + lr;
            const int d0 = M::dim(kb, grp, 0);
            window_to_lds16(vwin, buf + f * 1024,
                            d0 < ld ? (uint32_t)((row * ld + d0) * (int)sizeof(T)) : kDeadOffset);
        }
        const int g = min(ngroups - 1, cb * GPB + (PARTS == 1 ? wave : wave >> 1));
        const int q = min(kt - 1, is_r * PARTS + (PARTS == 1 ? 0 : wave & 1));
        const unsigned char *tile = tiles + ((int64_t)g * kt + q) * tbytes + HDR + (int64_t)is_k * 4096;
        const auto bwin = window_rsrc(tile, (uint32_t)(min(2, nkb - is_k * 2) * 2048));
#pragma unroll
        for (int i = 0; i < 4; ++i)
            window_to_lds16(bwin, buf + (4 * RT + wave * 4 + i) * 1024, (uint32_t)(i * 1024 + lane * 16));
        if (++is_k == ksteps) is_k = 0, ++is_r;
    };

    f32x4 acc[RT][2][NB], m[RT][2];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int s = 0; s < 2; ++s) m[rt][s] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};  // e0

    // The biases of round r's columns, the accumulators' seeds: a product
    // that comes close to |s|^2 then passes through sums of half its size
    // (added after the products, the error of f was up to 1.45 times that of
    // the kernel in bigd_kernels.hpp).
    float bias[2][NB];
    auto load_bias = [&](int r) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int g = min(ngroups - 1, cb * GPB + (PARTS == 1 ? wn * 2 + s : wn));
            const int q = min(kt - 1, r * PARTS + (PARTS == 1 ? 0 : s));
            const float *hb = reinterpret_cast<const float *>(tiles + ((int64_t)g * kt + q) * tbytes);
#pragma unroll
            for (int h = 0; h < NB; ++h) bias[s][h] = hb[h * 16 + lr];
        }
    };

    issue(0);
    load_bias(0);
    int st = 0;
    for (int r = 0; r < rounds; ++r) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int h = 0; h < NB; ++h)
                    acc[rt][s][h] = f32x4{bias[s][h], bias[s][h], bias[s][h], bias[s][h]};
        load_bias(r + 1);  // past the last round: its biases again
        for (int ks = 0; ks < ksteps; ++ks, ++st) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            issue(st + 1);  // past the last stage: its tiles again, never read
            const unsigned char *buf = smem + (st & 1) * SB;
            const vec_t *A = reinterpret_cast<const vec_t *>(buf) + wm * RT * 2 * 64 + lane;
            const vec_t *B = reinterpret_cast<const vec_t *>(buf + 4 * RT * 1024) + wn * 8 * 64 + lane;
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                vec_t b[2][NB], a[RT];
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int h = 0; h < NB; ++h) b[s][h] = B[(s * 4 + kb * 2 + h) * 64];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) a[rt] = A[(rt * 2 + kb) * 64];
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int s = 0; s < 2; ++s)
#pragma unroll
                        for (int h = 0; h < NB; ++h) acc[rt][s][h] = M::mma(a[rt], b[s][h], 0, acc[rt][s][h]);
            }
            // The next stage's copies, then six fragments ahead of the first
            // use and one more read after every three instructions (left
            // alone, the compiler reads a k-block's fragments in one burst:
            // 10^5 x 2 048, 1 024 sets of 16 bf16 6.24 ms against 5.57).
            __builtin_amdgcn_sched_group_barrier(0x020, AF + 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
            for (int i = 0; i < 2 * (RT + 4) - 6; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_group_barrier(0x008, 8 * RT, 0);
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    m[rt][s][i] = fmaxf(fmaxf(m[rt][s][i], acc[rt][s][0][i]), acc[rt][s][1][i]);
    }

    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the last copy

    // One partial sum per 32 points and set: the lane's eight values pairwise,
    // then the four groups of lanes.
    const int64_t G = (n + kWideRows - 1) / kWideRows;
#pragma unroll
    for (int s = 0; s < (PARTS == 1 ? 2 : 1); ++s) {
        const int g = cb * GPB + (PARTS == 1 ? wn * 2 + s : wn);
#pragma unroll
        for (int i = 0; i < RT / 2; ++i) {
            f32x4 x = m[2 * i][s], y = m[2 * i + 1][s];
            if (PARTS == 2)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[e] = fmaxf(x[e], m[2 * i][1][e]);
                    y[e] = fmaxf(y[e], m[2 * i + 1][1][e]);
                }
            float t = ((x[0] + y[0]) + (x[2] + y[2])) + ((x[1] + y[1]) + (x[3] + y[3]));
            t += __shfl_xor(t, 16);
            t += __shfl_xor(t, 32);
            const int64_t row = (row0 + wm * RT * 16) / kWideRows + i;
            if (grp == 0 && g < ngroups && row < G) partials[row * lpad + (int64_t)g * 16 + lr] = t;
        }
    }
}

template <typename T, int RT, int PARTS>
hipError_t wide_launch(const MfmaPlan &pl, const MfmaArgs &x, hipStream_t st) {
    auto kern = eval_wide_kernel<T, RT, PARTS>;
    constexpr int lds = 2 * wide_stage(RT);
    static std::atomic<bool> ready[kMaxDevices];  // the attribute holds for one device
    const int dev = current_device();
    if (dev < 0) return hipErrorInvalidDevice;
    if (!ready[dev].load(std::memory_order_acquire)) {
        const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        ready[dev].store(true, std::memory_order_release);
    }
    const int64_t nrb = (x.n + 2 * RT * 16 - 1) / (2 * RT * 16);
    const int64_t gpb = kWideStreams / PARTS, units = nrb * ((x.ngroups + gpb - 1) / gpb);
    if (units > (1 << 30) || x.ngroups > INT32_MAX || x.kt > INT32_MAX) return hipErrorInvalidValue;
    hipExtLaunchKernelGGL(kern, flat_grid((units + 7) / 8 * 8, kWideWaves * 64), dim3(kWideWaves * 64), lds, st, x.ev_start,
                          x.ev_stop, 0, (const T *)x.V, x.n, x.ld, pl.nkb, (const unsigned char *)x.tiles, (int)x.kt, (int)x.ngroups,
                          (int)nrb, x.partials, x.lpad);
    return hipGetLastError();
}

// The launch that finishes first: rounds of workgroups over the CUs, times
// the work of one (row tiles x member rounds; the factor is the LDS traffic
// per instruction, measured at d = 1 536).
template <typename T>
hipError_t wide_dispatch(const MfmaPlan &pl, const MfmaArgs &x, hipStream_t st) {
    const int64_t cus = std::max<int64_t>(1, device_cu_count());
    double best = 0.0;
    int rt = 0, parts = 0;
    for (int r : {8, 6, 4})
        for (int p : {1, 2}) {
            const int64_t units = ((x.n + 32 * r - 1) / (32 * r)) * ((x.ngroups * p + kWideStreams - 1) / kWideStreams);
            const double cost = (double)((units + cus - 1) / cus) * (double)((x.kt + p - 1) / p) * r *
                                (r == 8 ? 1.0 : r == 6 ? 1.05 : 1.2);
            if (rt == 0 || cost < best) best = cost, rt = r, parts = p;
        }
    if (parts == 1)
        return rt == 8 ? wide_launch<T, 8, 1>(pl, x, st) : rt == 6 ? wide_launch<T, 6, 1>(pl, x, st) : wide_launch<T, 4, 1>(pl, x, st);
    return rt == 8 ? wide_launch<T, 8, 2>(pl, x, st) : rt == 6 ? wide_launch<T, 6, 2>(pl, x, st) : wide_launch<T, 4, 2>(pl, x, st);
}

}  // namespace exemcl
