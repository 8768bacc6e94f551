// kernels_mfma.hip -- MFMA path planning and dispatch by storage type.  The
// kernels themselves are in mfma_kernels.hpp, instantiated per storage type
// in kernels_mfma_{f32,f16,bf16}.hip.
#include <stdlib.h>

#include "internal.h"
#include "mfma_kernels.hpp"
#include "split_kernels.hpp"
#include "wide_kernels.hpp"

// fp16/bf16 rows of at least EXEMCL_F16_WIDE_D coordinates use the 16x16x32
// shape.  Up to EXEMCL_HALF_MAX_D coordinates a last k-block of 16 covers
// d mod 32 in (0, 16] (d = 100: 3 x 32 + 16 = 112 instead of 128); above it
// d pads to whole 32-coordinate blocks (at most 8 % more work) and long tiles
// keep their cross-tile prefetch, which a half block does not take part in.
#ifndef EXEMCL_F16_WIDE_D
#define EXEMCL_F16_WIDE_D 17
#endif
#ifndef EXEMCL_HALF_MAX_D
#define EXEMCL_HALF_MAX_D 192
#endif
#ifndef EXEMCL_MAIN_MAX_D16
#define EXEMCL_MAIN_MAX_D16 1024
#endif
#ifndef EXEMCL_WIDE_MIN_N
#define EXEMCL_WIDE_MIN_N 6144
#endif
#if EXEMCL_HALF_MAX_D > 192
#error "half k-blocks are compiled for 2 to 6 k-blocks (d <= 192)"
#endif

namespace exemcl {

// k-block counts with a compiled kernel; d is zero-padded up to the next one.
static const int kBuckets[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 13, 14, 16, 20, 24, 28, 32};

static int bucket(int nkb) {
    for (int b : kBuckets)
        if (b >= nkb) return b;
    return -1;
}

// Largest d: the kernels address a block of rows through 32-bit byte
// offsets (32 rows of at most 2^24 fp32 coordinates).
constexpr int64_t kMaxD = int64_t(1) << 24;

// fp32 rows that fit the registers: whole blocks of 32 and the instructions
// of the tail (a tail that would take as many as a whole block, or one that
// is not compiled, is a zero-padded whole block).  d <= 2 stays on the fp32
// MFMA: one instruction holds all of it (10^5 points, 1 024 sets of 16: d = 2
// 90 us against 105 here; d = 4 137 against 104).
static bool split_plan(int64_t d, int64_t n, MfmaPlan *q) {
    if (d <= 2) return false;
    int nkb = (int)(d / 32), r4 = (int)(d % 32 + 3) / 4;
    int nt = (6 * r4 + 7) / 8;
    if (nt > (nkb <= 2 ? 4 : 3)) nkb += 1, nt = 0;
    // many whole blocks: one compiled tail
    if (nt > 0 && (nkb > 6 || (nkb == 6 && nt > 1))) nt = 3;
    if (split_steps(nkb, nt) > kSplitMaxSteps) return false;
    q->split = 1;
    q->d = (int)d;
    q->tile = kSplitSets;
    q->nb = 1;
    q->kb_dims = 32;
    q->nkb = nkb;
    q->nt = nt;
    q->rt = split_rt(nkb, nt, n);
    q->waves = kSplitWaves;
    q->rows = q->waves * q->rt * 16;
    q->wgsum = 1;
    return true;
}

int64_t split_charge(int64_t n, int64_t d, int64_t l, int64_t k) {
    const int64_t tm = split_charge_unit(d), groups = (l + tm - 1) / tm;
    const int64_t blocks = bucket((int)(tm == 32 ? (d + 7) / 8 : (d + 15) / 16));
    const int64_t waves = blocks <= 8 && tm == 32 ? 4 : 8;
    const int64_t rows = waves * (tm == 16 ? 16 : blocks <= 16 ? 64 : 32);
    auto up = [](int64_t x) { return (x + 255) / 256 * 256; };
    return up(up((n + rows - 1) / rows * waves * groups * tm * 4) +
              groups * k * ((blocks <= 4 && tm == 32 ? 256 : 128) + blocks * 1024));
}

int64_t split_charge_unit(int64_t d) { return d <= 256 ? 32 : 16; }

bool mfma_plan(int prec, int64_t d, int64_t n, MfmaPlan *p) {
    if (d < 1 || d > kMaxD) return false;
    MfmaPlan q{};
    if (prec == P_FP32 && split_plan(d, n, &q)) {
        *p = q;
        return true;
    }
    // fp16/bf16 up to d = 1024 stay on the register-resident kernel (one row
    // tile of 16 points and 32 k-blocks per wavefront); above that, and fp32
    // above 512, the coordinates are split over the wavefronts.
    const int64_t dmax_main = (prec == P_FP32) ? 512 : EXEMCL_MAIN_MAX_D16;
    if (d > dmax_main) {
        // Coordinates split over the 8 wavefronts of a workgroup sharing 32
        // points: 16x16x4 (fp32, 16 coordinates per k-block) or 16x16x32
        // (fp16/bf16, 32 per k-block, two members per tile); each wavefront
        // holds kw k-blocks per round, and d needs `rounds` rounds.
        q.bigd = 1;
        q.tile = 16;
        q.nb = prec == P_FP32 ? 1 : EXEMCL_NB16;
        q.kb_dims = prec == P_FP32 ? 16 : 32;
        q.nkb = (int)((d + q.kb_dims - 1) / q.kb_dims);
        q.nks_last = prec == P_FP32 ? 4 : 1;
        const int per = (q.nkb + 7) / 8;
        q.kw = per <= 2 ? 2 : per <= 4 ? 4 : 8;
        q.rounds = (q.nkb + 8 * q.kw - 1) / (8 * q.kw);
        q.rt = 2;
        q.waves = 8;
        q.rows = 32;
        if (prec != P_FP32 && d <= kWideMaxD && n >= EXEMCL_WIDE_MIN_N) {
            // A tiled product (wide_kernels.hpp): one partial sum per 32
            // points.  The line looks at n alone, since l and k must not
            // change a result's bits.  bf16, d = 1 536, coordinates split /
            // tiled: 6 144 points, 512 sets of 16 354 / 149 us, 64 sets of 8
            // 53 / 62 (too few blocks for the CUs); 12 288 points, d = 1 100,
            // 64 sets of 8 94 / 73.
            q.bigd = 0;
            q.wide = 1;
            q.wgsum = 1;
        }
        *p = q;
        return true;
    }
    q.waves = 4;
    q.nb = 1;
    q.half = 0;
    q.splat = 0;
    q.il = 0;
    if (prec == P_FP32) {
        // d <= 2: one v_mfma_f32_32x32x2_f32 holds both coordinates
        q.tile = 32;
        q.kb_dims = 8;
        q.nkb = 1;
        q.nks_last = 1;
        q.il = 1;
    } else if (d >= EXEMCL_F16_WIDE_D) {
        // v_mfma_f32_16x16x32_{f16,bf16}, 32 coordinates per k-block, two
        // set members per tile; when d mod 32 is in (0, 16] the last k-block
        // holds 16 coordinates (v_mfma_f32_16x16x16) instead of padding to 32
        q.tile = 16;
        q.kb_dims = 32;
        q.nkb = bucket((int)((d + 31) / 32));
        q.nks_last = 1;
        q.nb = EXEMCL_NB16;
        q.half = (d % 32 != 0 && d % 32 <= 16 && d <= EXEMCL_HALF_MAX_D && q.nkb == (d + 31) / 32) ? 1 : 0;
    } else {
        // v_mfma_f32_32x32x16_{f16,bf16}, 16 coordinates per k-block (one
        // k-block for d <= 16, where 32-coordinate blocks would be half padding)
        q.tile = 32;
        q.kb_dims = 16;
        q.nkb = bucket((int)((d + 15) / 16));
        q.nks_last = 1;
    }
    if (q.nkb < 1) return false;
    const int eb = prec == P_FP32 ? 4 : 2;
    q.rt = plan_rt(eb, q.tile, q.nkb);
    q.waves = plan_waves(eb, q.tile, q.nkb);
    q.rows = q.waves * q.rt * q.tile;
    q.splat = splat_bias(eb, q.tile, q.nkb) ? 1 : 0;
    q.wgsum = wg_sum(q.waves, q.nb) ? 1 : 0;
    *p = q;
    return true;
}

int64_t mfma_tile_bytes(const MfmaPlan &pl) {
    if (pl.split) return split_tile_bytes(pl.nkb, pl.nt);
    return hdr_bytes(pl.tile, pl.nb, pl.splat != 0) + (int64_t)(pl.nkb - pl.half) * pl.nb * 1024 +
           (int64_t)pl.half * pl.nb * 512;
}

bool mfma_gathers(int prec, const MfmaPlan &pl) {
    return pl.split || (prec != P_FP32 && !pl.bigd && !pl.wide && pl.nkb <= 4);
}

int64_t mfma_tiles_per_group(const MfmaPlan &pl, int64_t k) { return (k + pl.nb - 1) / pl.nb; }

hipError_t launch_pack(int prec, const MfmaPlan &pl, const void *V, int64_t n, int ld, const int32_t *sets,
                       int64_t l, int64_t k, void *tiles, hipStream_t st, const int32_t *live, int64_t live0) {
    if (pl.split) return split_pack_run(pl, V, n, ld, sets, l, k, tiles, st, live, live0);
    if (live) return hipErrorInvalidValue;
    switch (prec) {
    case P_FP32: return pack_run_f32(pl, V, n, ld, sets, l, k, tiles, st);
    case P_FP16: return pack_run_f16(pl, V, n, ld, sets, l, k, tiles, st);
    case P_BF16: return pack_run_bf16(pl, V, n, ld, sets, l, k, tiles, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_mfma(int prec, int mode, const MfmaPlan &pl, const void *V, int64_t n, int ld, const void *tiles,
                       int64_t kt, int64_t ngroups, int64_t gpc, const float *m0, float *partials, int64_t lpad,
                       float *rowmax, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop, const int32_t *sets,
                       int64_t l, int64_t k, const int32_t *live, int64_t live0, int m0_stride, int32_t *counter,
                       float *out, const void *E, int64_t ne) {
    const MfmaArgs x{V,    n, ld, tiles, kt, ngroups, gpc,   m0,        partials, lpad, rowmax,
                     sets, l, k,  E,     ne, live,    live0, m0_stride, counter,  out,  ev_start, ev_stop};
    if ((live || m0_stride != 1) && !(pl.split && m0 && tiles)) return hipErrorInvalidValue;
    if (!tiles && !(pl.split || (mfma_gathers(prec, pl) && mode == MODE_SUM && !m0))) return hipErrorInvalidValue;
    if (pl.bigd) return bigd_run(prec, mode, pl, x, st);
    if (pl.wide) return mode == MODE_SUM ? wide_run(prec, pl, x, st) : hipErrorInvalidValue;
    if (pl.split)
        return mode == MODE_ROWMAX ? (tiles ? split_rowmax_run(pl, x, st) : split_rowmax_gather_run(pl, x, st))
               : m0                ? (tiles ? split_gain_run(pl, x, st) : split_gain_gather_run(pl, x, st))
                                   : (tiles ? split_sum_run(pl, x, st) : split_gather_run(pl, x, st));
    switch (prec) {
    case P_FP32: return eval_run_f32(pl, mode, x, st);
    case P_FP16: return mode == MODE_SUM ? eval_run_f16(pl, mode, x, st) : hipErrorInvalidValue;
    case P_BF16: return mode == MODE_SUM ? eval_run_bf16(pl, mode, x, st) : hipErrorInvalidValue;
    }
    return hipErrorInvalidValue;
}

}  // namespace exemcl
