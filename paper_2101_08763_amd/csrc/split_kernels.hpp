// split_kernels.hpp -- fp32 evaluation on the bf16 matrix cores (templates;
// instantiated in kernels_mfma_split*.hip).
//
// The fp32 MFMA runs at a sixteenth of the bf16 rate and never overlaps VALU
// work.  An fp32 value is exactly the sum of three bf16 ones,
//     x = hi + mid + lo   (hi = bf16(x), mid = bf16(x - hi), lo = the rest),
// and of the nine products of two such sums six matter: each of the other
// three is at most 2^-25 of |x||y| (parts round to nearest, so |mid| <= 2^-8
// |x| and |lo| <= 2^-17 |x|), their sum at most 2^-24, one rounding of fp32,
// and of either sign.  So
//     <v, s> = sum  lo*hi + hi*lo + mid*mid + mid*hi + hi*mid + hi*hi
// on v_mfma_f32_16x16x32_bf16 (products exact, fp32 accumulation), six
// instructions of 32 coordinates where fp32 needs sixteen times their time.
// The five small products run in an accumulator of their own: added into the
// large one they lose their low bits there, always downwards.  Measured
// against 64 bits, random and clustered points, h_s(v) of d = 8 / 32 / 100 /
// 256 / 512 coordinates: rms error 3.6 / 4.8 / 8.3 / 15 / 21 e-8 of the
// values' rms, fp32 MFMA 6.7 / 14 / 24 / 43 / 60 e-8 (one accumulator for
// all six products: 5.3 / 12 / 20 / 36 / 46 e-8 and a mean of -4e-8).  f
// averages those errors away; what is left are the exemplars' norms and the
// sums over points, both summed in fp64 beyond short runs: rms error of f, 34
// values of d from 3 to 512, eval and gain, 0.38 to 1.00 times that of the
// fp32 MFMA kernels.
//
// Bound by the matrix cores (a sixth of the bf16 peak is 419 TFLOP/s; busy
// 83 % of the time at 50 000 x 100, 5 000 sets of 10) up to about 200
// coordinates.  Where one row tile is all the registers hold, a (half) tile is
// little work between two barriers (d = 512: matrix cores busy 68 % of the
// time, LDS reads 34 %).  A call, fp32 MFMA -> here: 50 000 x 100, 5 000 sets
// of 10 3 539 -> 1 809 us; 50 000 x 32, 256 sets of 10 78.3 -> 48.9; 30 011 x
// 301, 333 sets of 7 389 -> 194; the kernel at 10^5 points, 1 024 sets of 16:
// d = 16 132 -> 261 TFLOP/s, d = 128 142 -> 289, d = 512 133 -> 247.
//
// Everything else follows mfma_kernels.hpp: the clamp form, points resident
// in registers, exemplar tiles streamed through LDS, a running max per
// (point, set), no work matrix.  Differences:
//   - a tile is one member of 32 sets: two column groups of 16 sets, so an
//     odd or single member costs nothing;
//   - the d coordinates are NKB whole blocks of 32, three operand parts each,
//     and a tail of r = d - 32 NKB coordinates whose six products lie side by
//     side in the instruction's 32 places, in quads of four coordinates:
//     NT = 1, 2, 3, 3, 4 instructions for r <= 4, 8, 12, 16, 20 instead of
//     six (a longer tail is a zero-padded whole block);
//   - rows are read with 4-byte alignment, so V never needs a padded copy.
#pragma once

#include <algorithm>
#include <atomic>
#include <float.h>
#include <stdlib.h>

#include <hip/hip_ext.h>

#include "device.hpp"
#include "internal.h"
#include "mfma_kernels.hpp"

namespace exemcl {

// Tile header: 32 fp32 biases; without whole blocks four times each, so that
// a lane reads its four accumulators' seeds in one load.
constexpr int split_hdr(int nkb) { return nkb == 0 ? 512 : 128; }
constexpr int kSplitSets = 32;   // sets per tile
constexpr int kSplitMaxSteps = 48;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Fragments of one column group: lo, mid, hi of every whole block, the tail.
constexpr int split_steps(int nkb, int nt) { return 3 * nkb + nt; }
constexpr int split_tile_bytes(int nkb, int nt) { return split_hdr(nkb) + split_steps(nkb, nt) * 2048; }

__device__ __forceinline__ void split3(float x, __bf16 &hi, __bf16 &mid, __bf16 &lo) {
    hi = (__bf16)x;
    const float r = x - (float)hi;
    mid = (__bf16)r;
    lo = (__bf16)(r - (float)mid);
}

// The tail's places.  A lane holds 2 NT quads of places (quad 2 t + w: half w
// of fragment t); u = ceil(r / 4) quads of coordinates have six products each
// (0 lo*hi, 1 hi*lo, 2 mid*mid, 3 mid*hi, 4 hi*mid, 5 hi*hi, a point's part
// first), laid out so that a lane reads one quad of coordinates, or two:
//   u = 1, NT = 1: quad 0 in every group of lanes, products 2 grp + w;
//   u = 2, NT = 2: quad grp / 2, products 4 t + 2 (grp % 2) + w;
//   u = 3 or 4, NT = 3: quad grp, products 2 t + w;
//   u = 5, NT = 4: as NT = 3, then in t = 3 products 2 grp + w of quad 4.
// A quad's small products come in earlier fragments than its hi*hi, or in the
// same one.  Products above 5 are zero.  (The bias -||s||^2/2 as three bf16
// parts in a free quad saves the accumulators' seeds, but beside hi*hi in one
// instruction it is truncated: results 3e-8 too small at d <= 12, against
// 0.1e-8 from the seeds.)
template <int NT>
struct Tail {
    static constexpr int OWN = 0, FIFTH = 1;  // which quad of coordinates
    // the first coordinate of the lane's own quad
    __device__ static int own(int grp) { return NT == 1 ? 0 : NT == 2 ? 4 * (grp >> 1) : 4 * grp; }
    // product of place quad (t, w)
    __device__ static int prod(int grp, int t, int w) {
        if (NT == 1) return 2 * grp + w;
        if (NT == 2) return 4 * t + 2 * (grp & 1) + w;
        return t < 3 ? 2 * t + w : 2 * grp + w;
    }
    static constexpr int which(int t) { return NT == 4 && t == 3 ? FIFTH : OWN; }
    // the first fragment that holds hi*hi of any quad
    static constexpr int BIG = NT == 4 ? 2 : NT - 1;
};

// A quad of coordinates as its three bf16 parts.
struct Quad {
    bf16x4 hi, mid, lo;
};
__device__ __forceinline__ Quad split_quad(const float (&x)[4]) {
    Quad q;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        __bf16 h, m, l;
        split3(x[e], h, m, l);
        q.hi[e] = h;
        q.mid[e] = m;
        q.lo[e] = l;
    }
    return q;
}
__device__ __forceinline__ u32x2 pick(int prod, const bf16x4 &p0, const bf16x4 &p1, const bf16x4 &p2, const bf16x4 &p3,
                                      const bf16x4 &p4, const bf16x4 &p5) {
    const u32x2 zero = {0u, 0u};
    auto b = [](const bf16x4 &x) { return __builtin_bit_cast(u32x2, x); };
    return prod == 0   ? b(p0)
           : prod == 1 ? b(p1)
           : prod == 2 ? b(p2)
           : prod == 3 ? b(p3)
           : prod == 4 ? b(p4)
           : prod == 5 ? b(p5)
                       : zero;
}
// Coordinates c .. c + 3 of the row at element `row` of a window, c a multiple
// of 4, zero from d on, in one load: the last quad of rows with d % 4 != 0 is
// read from its end and shifted (d >= 4).
__device__ __forceinline__ f32x4 window_quad(__amdgpu_buffer_rsrc_t rsrc, int row, int c, int d) {
    const int part = d & 3;
    const bool whole = c + 4 <= d;
    const f32x4 v = window_load16<f32x4>(rsrc, c < d ? (uint32_t)((row + (whole ? c : d - 4)) * 4) : kDeadOffset);
    if (part == 0) return v;
    f32x4 x = {part == 3 ? v[1] : part == 2 ? v[2] : v[3], part == 3 ? v[2] : part == 2 ? v[3] : 0.0f,
               part == 3 ? v[3] : 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = whole ? v[e] : x[e];
    return x;
}

// One lane's tail fragment t, of a point or of an exemplar.
template <int NT>
__device__ __forceinline__ bf16x8 tail_fragment(const Quad *q, int grp, int t, bool point) {
    const Quad &c = q[Tail<NT>::which(t)];
    u32x4 v;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const int prod = Tail<NT>::prod(grp, t, w);
        const u32x2 x = point ? pick(prod, c.lo, c.hi, c.mid, c.mid, c.hi, c.hi)
                              : pick(prod, c.hi, c.lo, c.mid, c.hi, c.mid, c.hi);
        v[2 * w] = x[0];
        v[2 * w + 1] = x[1];
    }
    return __builtin_bit_cast(bf16x8, v);
}

// One column group of one tile: lane L stages row `idx` of V (16 rows, lane
// L % 16 of each group of lanes) and their biases -||s||^2/2 to `tile`.
// ||s||^2 in fp64 (the lane's blocks and tail in order, then the four groups
// of lanes with a fixed xor tree), but for a block's eight coordinates where
// there are many blocks: its error is the same for every point and does not
// average out in f.  An invalid index is a zero column with bias -FLT_MAX,
// which never wins the running max.  Four whole blocks are loaded before any
// is stored; one at a time with few registers to spare (LEAN).
template <int NKB, int NT, bool LEAN = false>
__device__ __forceinline__ void stage_columns(const float *__restrict__ V, int64_t n, int ld, int d, int64_t idx,
                                              int h, int lane, unsigned char *tile) {
    const int grp = lane >> 4;
    const bool valid = idx >= 0 && idx < n;
    const float *row = V + (valid ? idx : 0) * (int64_t)ld;
    bf16x8 *dst = reinterpret_cast<bf16x8 *>(tile + split_hdr(NKB)) + h * 64 + lane;
    double sq = 0.0;
    constexpr int NQ = NT == 4 ? 2 : 1;  // quads of the tail the lane reads
    float xt[NQ][4];
    const int r = d - 32 * NKB;  // coordinates of the tail
    if constexpr (NT > 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int c0 = q == 0 ? Tail<NT>::own(grp) : 16;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool in = valid && c0 + e < r;
                const float x = row[in ? 32 * NKB + c0 + e : 0];
                xt[q][e] = in ? x : 0.0f;
            }
        }
    }
    constexpr int BATCH = LEAN ? 1 : 4, UNROLL = LEAN ? 1 : 16;
#pragma unroll UNROLL
    for (int k0 = 0; k0 < NKB; k0 += BATCH) {
        float x[BATCH][8];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            if (k0 + u >= NKB) continue;
            const int d0 = (k0 + u) * 32 + grp * 8;
            if ((k0 + u + 1) * 32 <= d) {
                const f32x4 a = *reinterpret_cast<const f32x4u *>(row + d0);
                const f32x4 b = *reinterpret_cast<const f32x4u *>(row + d0 + 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[u][e] = a[e], x[u][4 + e] = b[e];
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float v = row[d0 + e < d ? d0 + e : 0];
                    x[u][e] = d0 + e < d ? v : 0.0f;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            if (k0 + u >= NKB) continue;
            bf16x8 p[3];
            float b = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float v = valid ? x[u][e] : 0.0f;
                __bf16 hi, mid, lo;
                split3(v, hi, mid, lo);
                p[0][e] = lo;
                p[1][e] = mid;
                p[2][e] = hi;
                if constexpr (NKB < 4) sq = fma((double)v, (double)v, sq);
                else b = fmaf(v, v, b);
            }
            sq += (double)b;
#pragma unroll
            for (int q = 0; q < 3; ++q) dst[(NT + (k0 + u) * 3 + q) * 128] = p[q];
        }
    }
    if constexpr (NT > 0) {
        // every coordinate once: one lane group of those that read a quad
        const bool first = NT == 1 ? grp == 0 : NT == 2 ? (grp & 1) == 0 : true;
#pragma unroll
        for (int e = 0; e < 4; ++e) sq = fma((double)(first ? xt[0][e] : 0.0f), (double)xt[0][e], sq);
        if constexpr (NT == 4)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                sq = fma((double)(grp == 0 ? xt[NQ - 1][e] : 0.0f), (double)xt[NQ - 1][e], sq);
    }
    sq += __shfl_xor(sq, 16);
    sq += __shfl_xor(sq, 32);
    const float bias = valid ? (float)(-0.5 * sq) : -FLT_MAX;
    if constexpr (split_hdr(NKB) > 128) {
        if (grp == 0) reinterpret_cast<f32x4 *>(tile)[h * 16 + (lane & 15)] = f32x4{bias, bias, bias, bias};
    } else {
        if (grp == 0) reinterpret_cast<float *>(tile)[h * 16 + (lane & 15)] = bias;
    }
    if constexpr (NT > 0) {
        Quad q[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) q[i] = split_quad(xt[i]);
#pragma unroll
        for (int t = 0; t < NT; ++t)
            dst[t * 128] = tail_fragment<NT>(q, grp, t, false);
    }
}

// Staging: one workgroup of two wavefronts per tile (set group g, member p),
// one column group each; tile g*k + p at tiles + (g*k + p) * tile bytes.
// `live`: only *live - live0 of the l sets are there (counted on the device).
// `sets2`: after those, l2 sets of one member to tiles2.
template <int NKB, int NT>
__global__ __launch_bounds__(128) void pack_split_kernel(const float *__restrict__ V, int64_t n, int ld, int d,
                                                         const int32_t *__restrict__ sets, int64_t l, int64_t k,
                                                         unsigned char *__restrict__ tiles,
                                                         const int32_t *__restrict__ live, int64_t live0,
                                                         const int32_t *__restrict__ sets2, int64_t l2,
                                                         unsigned char *__restrict__ tiles2) {
    int64_t t = flat_block();
    if (sets2) {
        const int64_t first = (l + kSplitSets - 1) / kSplitSets * k;
        if (t >= first) t -= first, sets = sets2, l = l2, k = 1, tiles = tiles2;
    }
    const int64_t g = t / k, p = t - (t / k) * k;
    if (g * kSplitSets >= l) return;
    if (live) {
        l = min(l, (int64_t)*live - live0);
        if (g * kSplitSets >= l) return;
    }
    const int lane = threadIdx.x & 63, h = threadIdx.x >> 6;
    const int64_t j = g * kSplitSets + h * 16 + (lane & 15);
    const int64_t idx = j < l ? (int64_t)sets[j * k + p] : -1;
    stage_columns<NKB, NT>(V, n, ld, d, idx, h, lane, tiles + t * (int64_t)split_tile_bytes(NKB, NT));
}

// Stage geometry: as many tiles as two buffers (and the partial sums) hold,
// at most kSplitTpsMax; a workgroup of at most 4 wavefronts leaves room for
// a second one on the CU.
constexpr int kSplitLds = 160 * 1024;
constexpr int kSplitTpsMax = 8;
constexpr int split_round(int bytes, int waves) { return (bytes + waves * 1024 - 1) / (waves * 1024) * (waves * 1024); }
constexpr int split_budget(int waves) { return waves >= 8 ? kSplitLds : kSplitLds / (waves >= 4 ? 2 : 4); }
constexpr int split_red_bytes(int tps, int waves) { return 2 * tps * waves * 32 * 4; }
constexpr int split_tps(int nkb, int nt, int waves) {
    int tps = kSplitTpsMax;
    while (tps > 1 && 2 * split_round(tps * split_tile_bytes(nkb, nt), waves) + split_red_bytes(tps, waves) > split_budget(waves))
        --tps;
    return tps;
}
// Tiles of which two do not fit (d above 352) are staged in two halves, each
// with a buffer of its own; `gather` stages such a tile whole in one buffer.
constexpr bool split_halves(int nkb, int nt, int waves) {
    return 2 * split_round(split_tile_bytes(nkb, nt), waves) + split_red_bytes(1, waves) > kSplitLds;
}
constexpr int split_first(int nkb, int nt) { return split_hdr(nkb) + (split_steps(nkb, nt) + 1) / 2 * 2048; }
constexpr int split_stage_bytes(int nkb, int nt, int waves, bool gather) {
    return split_round(split_halves(nkb, nt, waves) && !gather ? split_first(nkb, nt)
                                                               : split_tps(nkb, nt, waves) * split_tile_bytes(nkb, nt),
                       waves);
}
// The points' parts leave no registers to stage in beside them: `gather` then
// has one buffer, and reads the points again for every stage.
constexpr bool split_reload(int nkb, bool gather) { return gather && nkb > 4; }
constexpr int split_buffers(int nkb, int nt, int waves, bool gather) {
    return gather && (split_halves(nkb, nt, waves) || split_reload(nkb, gather)) ? 1 : 2;
}
constexpr int split_lds(int nkb, int nt, int waves, bool gather) {
    return split_buffers(nkb, nt, waves, gather) * split_stage_bytes(nkb, nt, waves, gather) +
           split_red_bytes(split_tps(nkb, nt, waves), waves);
}

// Row tiles per wavefront: as many as the registers hold without spilling in
// the main loop (3 operand fragments per whole block and row tile).  A
// smaller ground set takes fewer: row blocks for all CUs, and less to load
// and split before the first product.  The rule looks at n and never at l or
// k, which must not change a result; so each line is a mean of long and short
// calls (256 sets of 10, 64 of 4, microseconds):
//   d = 8    700 points   1 or 2: 11.5, 11.5    4: 12.6, 11.4
//          7 000          1: 14.0, 11.4         2: 11.7, 11.5    4: 12.9, 11.5
//         20 000          2: 17.4, 11.4         4: 17.6, 11.4
//         40 000          2: 23.5, 14.1         4: 21.7, 11.4
//   d = 40   4 000        1: 15.8, 12.7         2: 17.5, 12.8
//         12 000          1: 26.0, 12.8         2: 25.1, 13.0    4: 23.5, 16.3
//         30 000          2: 40.0, 13.3         4: 36.6, 17.2
//         64 000          2: 68.2, 17.9         4: 62.2, 18.0
//         80 000          2: 88.0, 22.7         4: 79.9, 22.4
//   d = 100  4 000        1: 21.0, 15.2         2: 26.7, 18.5
//         12 000          1: 42.9, 16.4         2: 42.8, 19.2    3: 38.4, 24.0
//         30 000          2: 73.7, 19.7         3: 77.8, 26.7
//         40 000          2: 96.8, 24.7         3: 94.0, 27.6
//         80 000          2: 178, 37.1          3: 172, 32.1
// Up to 65 536 points two row tiles are one round of workgroups.
constexpr int kSplitWaves = 8;
constexpr int split_rt_max(int nkb, int nt) {
    const int steps = split_steps(nkb, nt);
    return steps <= 5 ? 4 : steps <= 10 ? 3 : steps <= 19 ? 2 : 1;
}
constexpr int split_rt(int nkb, int nt, int64_t n) {
    const int top = split_rt_max(nkb, nt);
    if (top == 1) return 1;
    if (nkb == 0) return n < 1024 ? 1 : n < 32768 ? 2 : top;
    return n < 8192 ? 1 : n < (top == 4 ? 65537 : 32768) ? 2 : top;
}
// The cache g(v) reads V once against a few tiles: small workgroups, of two
// row tiles; one row tile and eight wavefronts where the registers hold one,
// since a tile's LDS then leaves room for a single workgroup on the CU
// (20 000 x 512, 7 points: 20.6 us; two row tiles, which spill, and four
// wavefronts 45.6).
constexpr int split_rowmax_rt(int nkb, int nt) { return std::min(2, split_rt_max(nkb, nt)); }
constexpr int split_rowmax_waves(int nkb, int nt) { return split_rt_max(nkb, nt) == 1 ? 8 : 4; }

// ---------------------------------------------------------------------------
// Evaluation.  A workgroup owns WAVES*RT*16 consecutive points; units of work
// are (row block, set group) pairs, shared out as in mfma_kernels.hpp: S
// workgroups take the whole row blocks w, w + S, ... first (all walk the set
// groups in step, so the tiles stay in L2), then equal contiguous shares of
// the units of the rest.
//
// MODE_SUM: partials[rb * lpad + j] = sum over the row block's points of
// max(m0(v), max_p h_{s_jp}(v)); wavefront sums go to LDS as set groups end.
// When the next stage could fill their half of the buffer they are added, in a
// fixed order, after its barrier: in fp64, like the second pass, since the
// seven roundings of fp32 sums are up to 13 % of the error of f at small d
// (d = 4: 3.5e-8 rms against 3.3e-8), and many at a time, by all wavefronts,
// since the others wait for the one that adds (after every stage: 50 000 x 16,
// 1 024 sets of 8 67.7 us against 66.1).
// MODE_ROWMAX: rowmax[v] = max(m0(v), 0, max over all staged columns of
// h_s(v)); rowmax may be m0 (a point is read and written by one workgroup).
//
// GATHER: no staged tiles in memory; the workgroup stages every tile into LDS
// itself, from the set indices, with the same code and so the same bits.
// `tiles` is then the matrix those indices address (rows of `ld`, like V's),
// and `live0` its number of rows.
// ---------------------------------------------------------------------------
template <int NKB, int NT, int RT, int WAVES, int MODE, bool HAS_M0, bool GATHER>
__global__ __launch_bounds__(WAVES * 64, 2) void eval_split_kernel(
    const float *__restrict__ V, int64_t n, int ld, int d, const unsigned char *__restrict__ tiles, int64_t kt,
    int64_t ngroups, int64_t nrb, const float *m0, float *partials, int64_t lpad, float *rowmax,
    const int32_t *__restrict__ sets, int64_t l, const int32_t *__restrict__ live, int64_t live0, int m0_stride,
    int32_t *counter, float *__restrict__ out) {
    if constexpr (HAS_M0 && MODE == MODE_SUM && !GATHER) {
        // scoring a list whose length was counted on the device
        if (live) {
            const int64_t cnt = (int64_t)*live - live0;
            if (cnt <= 0) return;
            ngroups = min(ngroups, (cnt + kSplitSets - 1) / kSplitSets);
        }
    }
    constexpr int STEPS = split_steps(NKB, NT);
    constexpr int TB = split_tile_bytes(NKB, NT);
    constexpr int TPS = split_tps(NKB, NT, WAVES);
    constexpr int NTHR = WAVES * 64;
    constexpr int NBUF = split_buffers(NKB, NT, WAVES, GATHER);
    constexpr bool RELOAD = split_reload(NKB, GATHER);
    constexpr int SB = split_stage_bytes(NKB, NT, WAVES, GATHER);
    constexpr int CNT = SB / (NTHR * 16);
    // HALF: a stage is half a tile (HSTEPS steps, HBYTES bytes, then the rest)
    constexpr bool HALF = split_halves(NKB, NT, WAVES) && !GATHER;
    constexpr int HSTEPS = HALF ? (STEPS + 1) / 2 : STEPS, HBYTES = split_first(NKB, NT);
    static_assert(NBUF * SB + split_red_bytes(TPS, WAVES) <= kSplitLds, "LDS");
    constexpr int PF = STEPS == 1 || STEPS > 42 ? 1 : 2;  // steps of B fragments read ahead
    // Above 36 steps every register counts: the copies' offsets are computed
    // for every stage (kept, they spilled points' parts, whose reloads wait
    // for the copies: 100 000 x 512, 1 024 sets of 16 10.1 ms, 6.8 now).
    constexpr bool TIGHT = STEPS > 36;
    constexpr int ROWS = WAVES * RT * 16;
    // An accumulator for the small products; the few of a tail alone go onto
    // the bias one after the other (error above), which saves the additions.
    constexpr bool SMALL = NKB > 0;
    constexpr int BIG = Tail<NT>::BIG;
    constexpr int HDR = split_hdr(NKB);
    // Short tiles: the fold of the running max is the busiest unit.
    constexpr bool PAIR = NKB == 0 && MODE == MODE_SUM && !HAS_M0;
    // Scoring S u {c}: sets of one member, whose maximum with the cached
    // value is summed as it comes; no running max is kept.
    constexpr bool ONE = HAS_M0 && MODE == MODE_SUM;

    extern __shared__ __align__(16) unsigned char smem[];
    float *red = reinterpret_cast<float *>(smem + NBUF * SB);

    auto segment = [&](const int64_t rb, const int64_t g0, const int64_t g1) {
        // hidden per segment, so that per-lane offsets are not kept in
        // registers through the whole persistent loop
        int tid = threadIdx.x, ldv = ld;
        asm volatile("" : "+v"(tid), "+s"(ldv));
        const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int lr = lane & 15, grp = lane >> 4;

        const int64_t ntiles = (g1 - g0) * kt;
        const int nst = (int)((ntiles + TPS - 1) / TPS);
        const unsigned char *chunk = tiles + g0 * kt * (int64_t)TB;
        const int64_t chunk_bytes = ntiles * (int64_t)TB;

        // Stage s into its buffer (HALF: half s % 2 of tile s / 2).
        auto issue = [&](int s) {
            unsigned char *buf = smem + (NBUF > 1 ? s & 1 : 0) * SB;
            if constexpr (GATHER) {
                const int tn = (int)min((int64_t)TPS, ntiles - (int64_t)s * TPS);
                for (int c = wave; c < 2 * tn; c += WAVES) {  // column group c % 2 of tile c / 2
                    const int64_t t = (int64_t)s * TPS + (c >> 1);
                    const int64_t g = t / kt, q = t - g * kt;
                    const int64_t j = (g0 + g) * kSplitSets + (c & 1) * 16 + lr;
                    const int64_t idx = j < l ? (int64_t)sets[j * kt + q] : -1;
                    stage_columns<NKB, NT, RELOAD>(reinterpret_cast<const float *>(tiles), live0, ldv, d, idx, c & 1,
                                                      lane, buf + (c >> 1) * TB);
                }
                return;
            }
            const int64_t base = HALF ? (s >> 1) * (int64_t)TB + (s & 1) * HBYTES : s * (int64_t)(TPS * TB);
            const int64_t most = HALF ? (s & 1 ? TB - HBYTES : HBYTES) : TPS * TB;
            const auto win = window_rsrc(chunk + base, (uint32_t)min(most, chunk_bytes - base));
            int at = tid * 16;
            if constexpr (TIGHT) asm volatile("" : "+v"(at));
#pragma unroll
            for (int r = 0; r < CNT; ++r)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    win, (__attribute__((address_space(3))) void *)(buf + (r * NTHR + wave * 64) * 16), 16,
                    at + r * NTHR * 16, 0, 0, 0);
        };
        if (nst > 0) issue(0);
        if (NBUF > 1 && (HALF || nst > 1)) issue(1);

        // This wavefront's points in A-operand order: three parts of every
        // whole block, the tail's places.  Rows past n read as zeros.
        const int64_t wrow0 = rb * (int64_t)ROWS;
        const int64_t wrows = min((int64_t)ROWS, n - wrow0);
        const auto vwin = window_rsrc(V + wrow0 * (int64_t)ldv, (uint32_t)(wrows * ldv * 4));
        bf16x8 a[RT][NKB > 0 ? NKB : 1][3], at[RT][NT > 0 ? NT : 1];
        auto load_points = [&]() {
            int row = lr;
            if constexpr (RELOAD) asm volatile("" : "+v"(row));  // loads of its own for every stage
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const int rowoff = (wave * RT * 16 + rt * 16 + row) * ldv;
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) {
                    const int d0 = kb * 32 + grp * 8;
                    f32x4 p, q;
                    if ((kb + 1) * 32 <= d) {
                        p = window_load16<f32x4>(vwin, (uint32_t)((rowoff + d0) * 4));
                        q = window_load16<f32x4>(vwin, (uint32_t)((rowoff + d0 + 4) * 4));
                    } else {
                        p = window_quad(vwin, rowoff, d0, d);
                        q = window_quad(vwin, rowoff, d0 + 4, d);
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        __bf16 hi, mid, lo;
                        split3(e < 4 ? p[e & 3] : q[e & 3], hi, mid, lo);
                        a[rt][kb][0][e] = lo;
                        a[rt][kb][1][e] = mid;
                        a[rt][kb][2][e] = hi;
                    }
                }
                if constexpr (NT > 0) {
                    constexpr int NQ = NT == 4 ? 2 : 1;
                    Quad q[NQ];
#pragma unroll
                    for (int i = 0; i < NQ; ++i) {
                        const int c0 = 32 * NKB + (i == 0 ? Tail<NT>::own(grp) : 16);
                        float x[4];
                        if (NKB == 0 && NT == 1 && d < 4) {  // d = 3
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                x[e] = window_load4(vwin, e < d ? (uint32_t)((rowoff + e) * 4) : kDeadOffset);
                        } else {
                            const f32x4 v = window_quad(vwin, rowoff, c0, d);
#pragma unroll
                            for (int e = 0; e < 4; ++e) x[e] = v[e];
                        }
                        q[i] = split_quad(x);
                    }
#pragma unroll
                    for (int t = 0; t < NT; ++t) at[rt][t] = tail_fragment<NT>(q, grp, t, true);
                }
            }
        };
        if constexpr (!RELOAD) load_points();

        // Initial running max: e0's 0, or the cached per-point value.
        float minit[HAS_M0 ? RT : 1][4];
        if constexpr (HAS_M0) {
            // m0 may be null in MODE_ROWMAX (an empty window reads as zeros)
            const auto mwin = window_rsrc(m0 ? m0 + wrow0 * m0_stride : V,
                                          m0 ? (uint32_t)(((wrows - 1) * m0_stride + 1) * 4) : 0u);
            if (m0_stride == 1 && wrows == ROWS) {  // whole quads
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const f32x4 v = window_load16<f32x4>(mwin, (uint32_t)((wave * RT * 16 + rt * 16 + 4 * grp) * 4));
#pragma unroll
                    for (int i = 0; i < 4; ++i) minit[rt][i] = v[i];
                }
            } else {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        minit[rt][i] =
                            window_load4(mwin, (uint32_t)((wave * RT * 16 + rt * 16 + 4 * grp + i) * m0_stride * 4));
            }
        }
        auto m_init = [&](int rt, int i) -> float {
            if constexpr (HAS_M0) return minit[rt][i];
            else return 0.0f;
        };
        float m[RT][2][4];
        auto m_reset = [&]() {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i) m[rt][h][i] = m_init(rt, i);
        };
        if constexpr (!ONE) m_reset();

        // B fragments (both column groups of a step) are read PF steps ahead
        // of use, across tiles of a stage.
        bf16x8 bq[PF][2];
        f32x4 bias[2];  // a column's bias, once per accumulator
        auto frag = [&](const unsigned char *tb, int s, int h) {
            const unsigned char *f = s < HSTEPS ? tb + HDR + s * 2048 : smem + SB + (s - HSTEPS) * 2048;
            return reinterpret_cast<const bf16x8 *>(f)[h * 64 + lane];
        };
        auto bias_of = [&](const unsigned char *tb, int h) {
            if constexpr (HDR > 128) return reinterpret_cast<const f32x4 *>(tb)[h * 16 + lr];
            const float b = reinterpret_cast<const float *>(tb)[h * 16 + lr];
            return f32x4{b, b, b, b};
        };
        auto head = [&](const unsigned char *tb) {
#pragma unroll
            for (int s = 0; s < PF; ++s)
#pragma unroll
                for (int h = 0; h < 2; ++h) bq[s][h] = frag(tb, s, h);
#pragma unroll
            for (int h = 0; h < 2; ++h) bias[h] = bias_of(tb, h);
        };
        // h_s(v) of one tile's 32 columns.
        // `mid`: called before the second half of the steps (HALF).
        auto tile = [&](const unsigned char *tb, const unsigned char *tnext, f32x4 (&acc)[RT][2], auto mid) {
            constexpr f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
            f32x4 sml[RT][2];
            f32x4 seed[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) seed[h] = bias[h];
#pragma unroll
            for (int s = 0; s < STEPS; ++s) {
                bf16x8 b[2];
                if (HALF && s == HSTEPS) {
                    mid();
#pragma unroll
                    for (int q = 0; q < PF; ++q)
#pragma unroll
                        for (int h = 0; h < 2; ++h) bq[q][h] = frag(tb, s + q, h);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    b[h] = bq[0][h];
#pragma unroll
                    for (int q = 0; q + 1 < PF; ++q) bq[q][h] = bq[q + 1][h];
                    if (s + PF < (s < HSTEPS ? HSTEPS : STEPS)) bq[PF - 1][h] = frag(tb, s + PF, h);
                    else if (!HALF) bq[PF - 1][h] = frag(tnext, s + PF - STEPS, h);
                    if (!HALF && s + PF == STEPS) bias[h] = bias_of(tnext, h);
                }
                __builtin_amdgcn_sched_barrier(0);
                auto mma = [](const bf16x8 &x, const bf16x8 &y, const f32x4 &c) {
                    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, c, 0, 0, 0);
                };
                if (s < NT) {
                    // fragments from BIG on hold hi*hi; the earlier ones
                    // small products only
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            if (SMALL && s < BIG)
                                sml[rt][h] = mma(at[rt][s], b[h], s == 0 ? zero : sml[rt][h]);
                            else
                                acc[rt][h] = mma(at[rt][s], b[h], s == (SMALL ? BIG : 0) ? seed[h] : acc[rt][h]);
                        }
                } else {
                    const int kb = (s - NT) / 3, part = (s - NT) % 3;  // exemplar part: lo, mid, hi
#pragma unroll
                    for (int q = 0; q <= part; ++q)  // point parts: hi | mid, hi | lo, mid, hi
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const bf16x8 &x = a[rt][kb][2 - part + q];
                                if (part == 2 && q == 2)
                                    acc[rt][h] = mma(x, b[h], NT == 0 && kb == 0 ? seed[h] : acc[rt][h]);
                                else
                                    sml[rt][h] = mma(x, b[h], kb == 0 && part == 0 && NT < 2 ? zero : sml[rt][h]);
                            }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (SMALL) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int i = 0; i < 4; ++i) acc[rt][h][i] += sml[rt][h][i];
            }
        };
        auto fold = [&](const f32x4 (&x)[RT][2]) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        m[rt][h][i] = fmaxf(ONE ? minit[HAS_M0 ? rt : 0][i] : m[rt][h][i], x[rt][h][i]);
        };
        auto fold2 = [&](const f32x4 (&x)[RT][2], const f32x4 (&y)[RT][2]) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int i = 0; i < 4; ++i) m[rt][h][i] = fmaxf(fmaxf(m[rt][h][i], x[rt][h][i]), y[rt][h][i]);
        };

        // Sums of the running maxima: this lane's, pairwise in a fixed order,
        // then the four groups of lanes (0 + 2, 1 + 3, then both).  Lanes
        // 0-15 end with the sums of column group 0, lanes 32-47 with those
        // of group 1.
        auto lane_sum = [&](int h) {
            constexpr int NV = RT * 4;
            float v[NV];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[rt * 4 + i] = m[rt][h][i];
#pragma unroll
            for (int c = NV; c > 1; c = (c + 1) / 2) {
                const int half = (c + 1) / 2;
#pragma unroll
                for (int i = 0; i + half < c; ++i) v[i] += v[i + half];
            }
            return v[0];
        };
        auto column_sums = [&]() {
            const float s0 = lane_sum(0), s1 = lane_sum(1);
            const float s = (lane < 32 ? s0 : s1) + __shfl_xor(lane < 32 ? s1 : s0, 32);
            return s + __shfl_xor(s, 16);
        };

        const int ktile = (int)kt;
        int p = 0;             // members of the current set group done
        int64_t gflush = g0;   // first set group whose sums are not stored yet
        int done = 0;          // set groups ended since, their sums in half `fill` of red
        int fill = 0;
        const int ends = (TPS - 1) / ktile + 1;  // set groups a stage may end
        auto flush = [&](int par, int cnt) {
            for (int i = tid; i < cnt * 32; i += NTHR) {
                const float *r = red + ((par * TPS + (i >> 5)) * WAVES) * 32 + (i & 31);
                double t[WAVES];
#pragma unroll
                for (int w = 0; w < WAVES; ++w) t[w] = (double)r[w * 32];
#pragma unroll
                for (int h = WAVES / 2; h >= 1; h /= 2)
#pragma unroll
                    for (int w = 0; w < h; ++w) t[w] += t[w + h];
                partials[rb * lpad + gflush * 32 + i] = (float)t[0];
            }
            gflush += cnt;
        };
        for (int s = 0; s < nst; ++s) {
            if (NBUF == 1 && s > 0) {
                __syncthreads();
                issue(s);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            const unsigned char *buf = smem + (HALF || NBUF == 1 ? 0 : s & 1) * SB;
            const int tn = (int)min((int64_t)TPS, ntiles - (int64_t)s * TPS);
            if constexpr (RELOAD) load_points();
            head(buf);
            if (NBUF > 1 && s > 0 && (HALF || s + 1 < nst)) issue(HALF ? 2 * s + 1 : s + 1);
            auto mid = [&]() {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                if (s + 1 < nst) issue(2 * (s + 1));
            };
            if (MODE == MODE_SUM && done + ends > TPS) {
                flush(fill, done);
                fill ^= 1;
                done = 0;
            }
            auto at_tile = [&](int i) { return buf + (i < tn ? i : tn - 1) * TB; };
            auto group_end = [&]() {
                const float t = column_sums();
                if (!(lane & 16)) red[((fill * TPS + done) * WAVES + wave) * 32 + (lane >> 5) * 16 + lr] = t;
                ++done;
                p = 0;
                if constexpr (!ONE) m_reset();
            };
            int i = 0;
            while (i < tn) {
                if constexpr (PAIR) {
                    // two members of the same sets: one max3 per element
                    while (i + 1 < tn && p + 1 < ktile) {
                        f32x4 x[RT][2], y[RT][2];
                        tile(at_tile(i), at_tile(i + 1), x, mid);
                        tile(at_tile(i + 1), at_tile(i + 2), y, mid);
                        fold2(x, y);
                        i += 2;
                        p += 2;
                        if (p == ktile && MODE == MODE_SUM) group_end();
                    }
                    if (i >= tn) break;
                }
                f32x4 x[RT][2];
                tile(at_tile(i), at_tile(i + 1), x, mid);
                fold(x);
                ++i;
                if (MODE == MODE_SUM && (ONE || ++p == ktile)) group_end();
            }
        }
        if constexpr (MODE == MODE_SUM) {
            __syncthreads();
            if (done > 0) flush(fill, done);
        } else {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float x = fmaxf(fmaxf(m[rt][0][i], m[rt][1][i]), 0.0f);
#pragma unroll
                    for (int off = 1; off < 16; off <<= 1) x = fmaxf(x, __shfl_xor(x, off));
                    const int64_t r = wrow0 + wave * RT * 16 + rt * 16 + 4 * grp + i;
                    if (lr == 0 && r < n) rowmax[r] = x;
                }
        }
    };

    const int64_t S = gridDim.x;
    const int64_t q = nrb / S;
    const int64_t U2 = (nrb - q * S) * ngroups;
    int64_t v = (int64_t)blockIdx.x * U2 / S;
    const int64_t v1 = ((int64_t)blockIdx.x + 1) * U2 / S;
    for (int64_t seg = 0;; ++seg) {
        int64_t rb, g0, g1;
        if (seg < q) {
            rb = seg * S + (int64_t)blockIdx.x;
            g0 = 0;
            g1 = ngroups;
        } else {
            if (v >= v1) break;
            rb = q * S + v / ngroups;
            g0 = v - (v / ngroups) * ngroups;
            g1 = min(ngroups, g0 + (v1 - v));
            v += g1 - g0;
        }
        // the previous segment's last stage and sums may still be read
        if (seg > 0) __syncthreads();
        segment(rb, g0, g1);
    }
    if constexpr (GATHER && MODE == MODE_SUM && !HAS_M0) {
        // `counter`: the workgroup that ends last adds the partial sums, in
        // the second pass's order (reduce_sets_kernel), and saves its launch.
        if (counter && last_workgroup(counter, (int)gridDim.x, reinterpret_cast<int *>(red))) {
            finish_sets<WAVES * 64>(partials, nrb, lpad, l, n, sets, kt, out, reinterpret_cast<double *>(smem));
            if (threadIdx.x == 0) atomicExch(counter, 0);
        }
    }
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
template <int NKB, int NT>
hipError_t split_pack_t(const void *V, int64_t n, int ld, int d, const int32_t *sets, int64_t l, int64_t k,
                        void *tiles, hipStream_t st, const int32_t *live, int64_t live0, const int32_t *sets2, int64_t l2,
                        void *tiles2) {
    const int64_t count = (l + kSplitSets - 1) / kSplitSets * k + (l2 + kSplitSets - 1) / kSplitSets;
    hipLaunchKernelGGL((pack_split_kernel<NKB, NT>), flat_grid(count, 128), dim3(128), 0, st, (const float *)V, n, ld, d,
                       sets, l, k, (unsigned char *)tiles, live, live0, sets2, l2, (unsigned char *)tiles2);
    return hipGetLastError();
}

// Workgroups of a persistent launch: one per slot, sharing the units out
// evenly, or a whole number per row block, so that none crosses into another
// one and loads and splits points twice.  Whichever ends first: tiles of the
// longest share, and kSplitStart instructions' worth of them per row block.
constexpr int kSplitStart = 200;
inline int64_t split_grid(int64_t nrb, int64_t ngroups, int64_t kt, int64_t slots, int mfmas_per_tile) {
    const int64_t even = std::min(nrb * ngroups, slots);
    if (nrb > slots || even % nrb == 0) return even;
    const int64_t per = std::min(ngroups, slots / nrb);
    const int64_t start = kSplitStart / mfmas_per_tile;
    const int64_t whole = (ngroups + per - 1) / per * kt + start;
    const int64_t shared = (nrb * ngroups + slots - 1) / slots * kt + 2 * start;
    return whole <= shared ? nrb * per : even;
}

template <int NKB, int NT, int RT, int WAVES, int MODE, bool HAS_M0, bool GATHER>
hipError_t split_launch(const MfmaPlan &pl, const MfmaArgs &x, hipStream_t st) {
    auto kern = eval_split_kernel<NKB, NT, RT, WAVES, MODE, HAS_M0, GATHER>;
    constexpr int lds = split_lds(NKB, NT, WAVES, GATHER);
    constexpr int rows = WAVES * RT * 16;
    static_assert(RT <= split_rt_max(NKB, NT), "the points' parts are held in registers");
    if (MODE == MODE_SUM && pl.rows != rows) return hipErrorInvalidValue;
    // Resident workgroups per CU, queried once per instantiation and device
    // (the LDS attribute holds for one device).
    static std::atomic<int> occ[kMaxDevices];
    const int dev = current_device();
    if (dev < 0) return hipErrorInvalidDevice;
    int per_cu = occ[dev].load(std::memory_order_relaxed);
    if (per_cu <= 0) {
        hipError_t e = hipSuccess;
        if (lds > 64 * 1024)
            e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e == hipSuccess)
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kern, WAVES * 64, lds);
        if (e != hipSuccess) return e;
        if (per_cu < 1) return hipErrorInvalidValue;
        occ[dev].store(per_cu, std::memory_order_relaxed);
    }
    const int64_t nrb = (x.n + rows - 1) / rows;
    const int64_t slots = (int64_t)per_cu * device_cu_count();
    if (slots < 1) return hipErrorInvalidDevice;
    // MODE_ROWMAX: a workgroup sees every set group of its row block.
    int64_t grid = MODE == MODE_ROWMAX ? nrb : nrb * x.ngroups;
    if (MODE == MODE_SUM && persistent_mode() != kPersistOff) grid = split_grid(nrb, x.ngroups, x.kt, slots, 2 * RT * (6 * NKB + NT));
    grid = std::min<int64_t>(grid, UINT32_MAX / (WAVES * 64));  // the workgroups share out what there is
    hipExtLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(WAVES * 64), lds, st, x.ev_start, x.ev_stop, 0,
                          (const float *)x.V, x.n, x.ld, pl.d,
                          (const unsigned char *)(!GATHER ? x.tiles : x.E ? x.E : x.V), x.kt, x.ngroups, nrb, x.m0,
                          x.partials, x.lpad, x.rowmax, x.sets, x.l, x.live, !GATHER ? x.live0 : x.E ? x.ne : x.n,
                          x.m0_stride, x.counter, x.out);
    return hipGetLastError();
}

template <int NKB, int NT, int MODE, bool HAS_M0, bool GATHER>
hipError_t split_eval_t(const MfmaPlan &pl, const MfmaArgs &x, hipStream_t st) {
    constexpr int TOP = split_rt_max(NKB, NT);
    if constexpr (MODE == MODE_ROWMAX) {
        return split_launch<NKB, NT, split_rowmax_rt(NKB, NT), split_rowmax_waves(NKB, NT), MODE, HAS_M0, GATHER>(pl, x, st);
    } else {
        if constexpr (TOP > 1)
            if (pl.rt == 1) return split_launch<NKB, NT, 1, kSplitWaves, MODE, HAS_M0, GATHER>(pl, x, st);
        if constexpr (TOP > 2)
            if (pl.rt == 2) return split_launch<NKB, NT, 2, kSplitWaves, MODE, HAS_M0, GATHER>(pl, x, st);
        return split_launch<NKB, NT, TOP, kSplitWaves, MODE, HAS_M0, GATHER>(pl, x, st);
    }
}

// One call per compiled (whole blocks, tail instructions).
#ifndef EXEMCL_SPLIT_CASES
#define EXEMCL_SPLIT_CASES(F)                                                                              \
    F(0, 1) F(0, 2) F(0, 3) F(0, 4) F(1, 0) F(1, 1) F(1, 2) F(1, 3) F(1, 4) F(2, 0) F(2, 1) F(2, 2) F(2, 3) \
    F(2, 4) F(3, 0) F(3, 1) F(3, 2) F(3, 3) F(4, 0) F(4, 1) F(4, 2) F(4, 3) F(5, 0) F(5, 1) F(5, 2) F(5, 3) \
    F(6, 0) F(6, 1) F(6, 3) F(7, 0) F(7, 3) F(8, 0) F(8, 3) F(9, 0) F(9, 3) F(10, 0) F(10, 3) F(11, 0)      \
    F(11, 3) F(12, 0) F(12, 3) F(13, 0) F(13, 3) F(14, 0) F(14, 3) F(15, 0) F(15, 3) F(16, 0)
#endif
constexpr int split_key(int nkb, int nt) { return nkb * 8 + nt; }

}  // namespace exemcl
