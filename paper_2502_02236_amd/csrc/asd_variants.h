// asd_variants.h -- kernel variants (host and device).
#pragma once

#include <stdint.h>

namespace asd {

// Two-pass kernel variants: 0 recomputes f(S) and the thermal field in the
// corrector; 1 stashes them from the predictor; 2 (handles with the
// demagnetising field only) recomputes them in kernels that take whole
// coarse cells and form the cells' spin sums for the next field evaluation.
constexpr int kPlainVariants = 3;
constexpr int kCellRowVariant = 2;

// Fused SC kernel variant: TXE lanes across x (64, 32 or 16), WAVES
// wavefronts, R column slots per lane, z planes per tile LZ (0: all).
// Extended tile TXE x TYE with TYE = WAVES R 64 / TXE; interior
// (TXE - 2) x (TYE - 2) x LZ.
struct FusedVariant {
    int txe, waves, rows, lz;
};

inline int fused_variant_count(bool fp64) { return fp64 ? 13 : 26; }

// Narrow tiles with short z-chunks serve lattices that leave the chip idle (every
// plane of a march waits for the one before), wide ones without chunks large
// batches (less recomputed halo, longer rows); fused_default picks by size.  The
// twelve-wave tiles filled a CU with one workgroup at three waves per SIMD.
inline FusedVariant fused_variant(bool fp64, int v)
{
    static const FusedVariant f32v[26] = {
        {32, 4, 1, 11}, {64, 4, 2, 0},  {16, 4, 2, 11}, {32, 8, 1, 11}, {32, 4, 1, 17},
        {32, 8, 1, 17}, {32, 8, 1, 0},  {32, 4, 2, 11}, {64, 8, 2, 17}, {16, 4, 1, 11},
        {16, 8, 1, 11}, {16, 8, 1, 0},  {32, 8, 2, 8},  {32, 12, 1, 0}, {64, 12, 1, 0},
        {16, 12, 1, 0}, {32, 12, 1, 11}, {32, 6, 1, 0},  {64, 8, 1, 0},  {64, 16, 1, 0},
        {64, 8, 1, 17}, {32, 4, 1, 6},  {32, 4, 1, 3},  {16, 4, 1, 3},  {32, 4, 1, 2},
        {32, 4, 1, 1}};
    static const FusedVariant f64v[13] = {{32, 4, 1, 11}, {64, 4, 2, 0},  {32, 8, 1, 17},
                                         {32, 4, 1, 0},  {32, 8, 1, 11}, {16, 4, 1, 11},
                                         {32, 4, 2, 11}, {32, 12, 1, 0}, {32, 12, 1, 11},
                                         {32, 4, 1, 6},  {32, 4, 1, 3},  {32, 4, 1, 2},
                                         {32, 4, 1, 1}};
    const int n = fused_variant_count(fp64);
    if (v < 0 || v >= n) v = 0;
    return fp64 ? f64v[v] : f32v[v];
}

// Fused L1_0 kernel variants (cell tiles, both sublattices per column).
inline int fused_l10_variant_count(bool fp64) { return fp64 ? 7 : 9; }

inline FusedVariant fused_l10_variant(bool fp64, int v)
{
    static const FusedVariant f32v[9] = {{32, 4, 1, 9}, {32, 4, 1, 0}, {32, 8, 1, 9}, {16, 4, 1, 9},
                                         {32, 8, 1, 0}, {32, 4, 1, 5}, {32, 4, 1, 3}, {32, 4, 1, 2},
                                         {32, 4, 1, 1}};
    static const FusedVariant f64v[7] = {{32, 4, 1, 9}, {32, 4, 1, 0}, {16, 4, 1, 9}, {32, 4, 1, 5},
                                         {32, 4, 1, 3}, {32, 4, 1, 2}, {32, 4, 1, 1}};
    const int n = fused_l10_variant_count(fp64);
    if (v < 0 || v >= n) v = 0;
    return fp64 ? f64v[v] : f32v[v];
}

// the SC step that has the ten Philox rounds compiled in
inline bool fused_ten_rounds(bool fp64, int txe, int rounds, bool zper)
{
    return !fp64 && txe == 64 && rounds == 10 && !zper;
}

// variants whose z-chunks the kernels with the demagnetising field take: thinner
// ones would need a partial-sum slot per chunk that a coarse cell meets
inline bool fused_demag_chunk(const FusedVariant &f) { return f.lz == 0 || f.lz >= 6; }

// Modelled time (us) of a step with variant f: n tiles of planes_all xy planes in
// all, the longest march planes long.  A tile's workgroups run in rounds of as many
// as fit the CUs (waves per SIMD in FP32: SC 4 for 64 lanes, else 3; L1_0 3; in FP64:
// 2 and 1); a plane of a round takes a fixed latency plus its waves' share of a CU,
// at least one wave's chain; a 64-lane tile's rows cost less per wave.
// SC: fitted to 22 (FP32) and 20 (FP64) lattices of 720 sites to 10.6M on MI355X: 8 %
// and 6 % rms; the variant picked is within 4 % of the fastest of the candidates on
// all but three (7, 8 and 17 %), where the former fixed choice (32 lanes, chunks of
// 11) was up to 2.0x (2.8x) slower (FP32 and FP64: 16 x 16 x 8 sites 9.1 -> 5.6 us and
// 19.2 -> 9.2 us, 64 x 64 x 20 11.3 -> 7.2 and 26.4 -> 14.0; FP32: four 400 x 200 x 33
// windows 118 -> 96).
// L1_0: 17 lattices of 240 sites to 3.7M: 5 % and 3 % rms, the pick within 9 %, where
// chunks of 9 planes were up to 2.8x (3.1x) slower (24 x 20 x 9 cells 29.8 -> 10.8 us
// and 56.1 -> 18.8; 100 x 100 x 20 33.7 -> 21.9 us in FP32; 260 x 156 x 27 in FP64
// 200 -> 162, in FP32 still chunks of 9).
struct FusedModel {
    double launch, wave, wave64, chain, latency;
    int simd, simd64;
    // another variant than the first of the list is taken where the model puts it
    // this far below: with less a few lattices came out slower than with the first
    // (FP64 SC 150 x 150 x 20 by 4 %, an FP32 step of 334 x 200 x 33 sites between two
    // regions' steps, whose launches leave the caches cold, by 13 %, FP32 L1_0 130 x
    // 156 x 27 by 1 %)
    double margin;
    // factor on tiles of eight wavefronts: in FP64 they came out 9 to 22 % above the
    // model beside the first of the list (32 lattices), and with the margin alone some
    // were slower than it (two systems of 304 x 92 x 44 sites 107 -> 112 us, 16 of 32 x
    // 32 x 32 52.5 -> 54.2) or than four wavefronts without chunks (35 of 160 x 93 x 39
    // 788, 708 so); with the factor the pick is at most 1 % slower than the first on 61
    double eight;
};

inline FusedModel fused_model(bool l10, bool fp64)
{
    if (l10)
        return fp64 ? FusedModel{2.2, 1.507, 1.507, 5.85, 0.0, 1, 1, 0.9, 1.0}
                    : FusedModel{3.3, 0.133, 0.133, 0.4, 2.32, 3, 3, 0.9, 1.0};
    return fp64 ? FusedModel{3.8, 0.25, 0.25, 0.85, 1.0, 2, 2, 0.9, 1.07}
                : FusedModel{3.5, 0.086, 0.061, 0.35, 0.345, 3, 4, 0.85, 1.0};
}

inline double fused_model_us(const FusedModel &m, const FusedVariant &f, double n, double planes_all,
                             double planes)
{
    const double wave = f.txe == 64 ? m.wave64 : m.wave;
    const int simd = f.txe == 64 ? m.simd64 : m.simd;
    const int per_cu = 4 * simd / f.waves < 1 ? 1 : 4 * simd / f.waves;
    const double waves = planes_all * f.waves / (n * planes);  // per tile, of its average march
    auto round = [&](double per) {
        const double t = wave * per * waves;
        return planes * ((t > m.chain ? t : m.chain) + m.latency);
    };
    const int64_t slots = 256 * (int64_t)per_cu, full = (int64_t)n / slots, rest = (int64_t)n - full * slots;
    const double t = m.launch + full * round(per_cu) + (rest > 0 ? round((double)((rest + 255) / 256)) : 0.0);
    return f.waves == 8 ? t * m.eight : t;
}

// the variants fused_default chooses from (one column per lane), the first of the
// table first
inline const int *fused_default_list(bool l10, bool fp64, int *count)
{
    static const int f32[] = {0, 25, 24, 22, 23, 21, 4, 3, 5, 18, 19};
    static const int f64[] = {0, 12, 11, 10, 9, 3, 4, 2};
    static const int l32[] = {0, 8, 7, 6, 5, 1};
    static const int l64[] = {0, 6, 5, 4, 3, 1};
    if (l10) {
        *count = fp64 ? (int)(sizeof l64 / sizeof l64[0]) : (int)(sizeof l32 / sizeof l32[0]);
        return fp64 ? l64 : l32;
    }
    *count = fp64 ? (int)(sizeof f64 / sizeof f64[0]) : (int)(sizeof f32 / sizeof f32[0]);
    return fp64 ? f64 : f32;
}

inline int fused_count(bool l10, bool fp64)
{
    return l10 ? fused_l10_variant_count(fp64) : fused_variant_count(fp64);
}

inline FusedVariant fused_pick(bool l10, bool fp64, int v)
{
    return l10 ? fused_l10_variant(fp64, v) : fused_variant(fp64, v);
}

inline void fused_tile_interior(bool fp64, int v, int *tx, int *ty, bool l10 = false)
{
    FusedVariant f = fused_pick(l10, fp64, v);
    *tx = f.txe - 2;
    *ty = f.waves * f.rows * 64 / f.txe - 2;
}

}  // namespace asd
