// Which configuration a GEMM launch takes (a predicted time per configuration, the cheapest wins) and which workgroup takes
// which tile.  Plain C++ (no HIP), so that both can be compiled and checked on their own.
//
// With t = tiles of the configuration, c compute units, r = ceil(t / c) rounds and n stages of K, a launch is predicted at
//     fixed + per_round r + n (stage time of the rounds + stage_tile t / c) + out_mb (MB of Y) + weights_mb (MB of W)
// microseconds.  The stage time of a round is stage_round.  Where a CU holds two workgroups, two rounds run side by side
// and take stage_round together; a last one that is alone takes stage_lone, about six tenths of it.  No coefficient
// is negative, so a prediction grows with M, N and K, also outside the shapes that were timed.
//
// The coefficients come from 2050 shapes (FP6: 2550, N from 16; M 8 or 17 .. 16384, N .. 28672, K 128 or 256 .. 14336, weights from HBM
// and in the memory-side cache), every configuration timed on every shape: least squares, then adjusted so that the choices,
// not the predictions, come out best.  On 400 further shapes the choice for FP6 is 1.1 % slower on average than the fastest
// configuration of the shape, 30 % at worst (3.8 % and 72 % by a table fitted to K >= 2048 without the bytes of Y and with negative
// coefficients: 1062 x 8576 x 128 18.4 us for 6.9, 7448 x 24416 x 512 160 for 111).  The register kernels for packed nibbles were
// fitted again later, to 675 shapes (below); on 500 others that table is 0.5 % behind the fastest, 14 % at worst.
#pragma once

#include <stdint.h>

namespace sr {

struct GemmConfig {
    int id, bm, bn;
    bool pairs;                                          // two workgroups per CU
    float fixed, per_round, stage_round, stage_lone, stage_tile, out_mb, weights_mb;
};

struct GemmShape {
    int64_t M, N, K;
    int stage;                                           // codes of K per stage
    float weight_bytes;                                  // per code
    int64_t cus;
};

constexpr int64_t gemm_tiles(const GemmConfig &c, const GemmShape &s) { return ((s.M + c.bm - 1) / c.bm) * ((s.N + c.bn - 1) / c.bn); }
constexpr int64_t gemm_rounds(const GemmConfig &c, const GemmShape &s) { return (gemm_tiles(c, s) + s.cus - 1) / s.cus; }

constexpr float gemm_cost(const GemmConfig &c, const GemmShape &s)
{
    const int64_t r = gemm_rounds(c, s);
    const float stages = (float)(s.K / s.stage);
    const float round_time = c.pairs ? (float)(r / 2) * c.stage_round + (float)(r & 1) * c.stage_lone : (float)r * c.stage_round;
    return c.fixed + c.per_round * (float)r + stages * (round_time + c.stage_tile * (float)gemm_tiles(c, s) / (float)s.cus) +
           c.out_mb * 2e-6f * (float)s.M * (float)s.N + c.weights_mb * 1e-6f * s.weight_bytes * (float)s.N * (float)s.K;
}

// The cheapest configuration but `skip`, if it is predicted at least 5 % faster than `base` (which stays otherwise: the
// predictions of two large tiles are as close as their errors).
template <int COUNT> constexpr const GemmConfig *gemm_cheapest(const GemmConfig (&configs)[COUNT], const GemmConfig *base,
                                                               const GemmConfig *skip, const GemmShape &s)
{
    const GemmConfig *best = base;
    float best_cost = .95f * gemm_cost(*base, s);
    for (const GemmConfig &c : configs)
        if (const float v = gemm_cost(c, s); &c != skip && v < best_cost) { best = &c; best_cost = v; }
    return best;
}

// ---- FP6 pipe (gemm_f6.hip) ------------------------------------------------------------------------------------------
constexpr GemmConfig kF6Configs[] = {
    {61, 256, 256, false, .544f, 5.021f, .458f, 0.f, .388f, .085f, .027f},      // eight waves of 128 x 64
    {72, 192, 256, false, 1.089f, 3.895f, .400f, 0.f, .335f, .089f, .065f},     // eight waves of 96 x 64
    {65, 256, 128, false, 2.117f, 2.326f, .337f, 0.f, .264f, .185f, .001f},       // eight waves of 64 x 64, a ninth for the hint
    {68, 128, 256, false, 2.153f, 2.385f, .336f, 0.f, .236f, .125f, .091f},     // eight waves of 64 x 64
    {67, 128, 128, true, 2.743f, .715f, .474f, .260f, .129f, .077f, .047f},     // four waves of 64 x 64
    {69, 128, 64, true, 2.658f, .645f, .402f, .214f, .049f, .138f, .066f},      // four waves of 64 x 32
    // operands straight into registers, K split over eight waves (gemm_f6_stream.hip)
    {64064, 64, 64, false, 1.536f, 1.934f, .122f, 0.f, .006f, .294f, .105f},
    {48064, 48, 64, false, 1.537f, 1.601f, .111f, 0.f, .001f, .431f, .093f},
    {48032, 48, 32, true, 2.048f, .349f, .144f, .085f, .012f, .505f, .088f},
    {32064, 32, 64, true, 2.191f, .319f, .185f, .090f, .005f, .434f, .108f},
    {32032, 32, 32, true, 2.086f, .239f, .117f, .069f, .008f, .542f, .095f},
    {16032, 16, 32, true, 1.952f, .151f, .080f, .048f, .007f, .941f, .124f},
    {16016, 16, 16, false, 2.192f, .298f, .030f, 0.f, .001f, .868f, .114f},
};
constexpr GemmShape f6_shape(int64_t M, int64_t N, int64_t K, int64_t cus) { return {M, N, K, 128, .75f, cus}; }
constexpr const GemmConfig *f6_config(const GemmShape &s)
{
    // between 256 x 256 and 256 x 128 tiles the cheaper schedule of whole rounds decides first (the small tile, which moves
    // more LDS bytes per product, with a handicap of 15 %)
    const GemmConfig *base = gemm_rounds(kF6Configs[0], s) * 100 <= gemm_rounds(kF6Configs[2], s) * 50 * 115 / 100 ? &kF6Configs[0] : &kF6Configs[2];
    return gemm_cheapest(kF6Configs, base, nullptr, s);
}

// ---- packed nibbles, M > 16 (gemm_prefill.hip) -------------------------------------------------------------------------
constexpr GemmConfig kPackedConfigs[] = {
    {14, 128, 128, true, 3.027f, 1.335f, 1.091f, .702f, .216f, .073f, .050f},   // four waves of 64 x 64
    {15, 256, 128, false, 1.807f, 3.329f, 1.053f, 0.f, .405f, .061f, .028f},    // eight waves of 64 x 64: while one wave of a
                                                                                // SIMD is held up issuing LDS or DMA
                                                                                // instructions, the other can issue MFMAs
    {17, 128, 64, true, 2.595f, .723f, .863f, .548f, .153f, .130f, .047f},      // eight waves of 32 x 32
    {18, 192, 128, false, 1.404f, 2.505f, 1.047f, 0.f, .270f, .097f, .035f},    // eight waves of 96 x 32
    {19, 64, 128, true, 2.622f, .650f, .874f, .554f, .146f, .128f, .058f},      // eight waves of 32 x 32
    // Two sets of four waves of 64 x 64, each with half of every stage, one workgroup per CU: two waves per SIMD on one
    // 128 x 128 tile without widening anything twice, and a ring of four stages instead of two, which weights from HBM
    // need.  512 x 4096 x 14336 60.6 -> 40.7 us, 190 x 9456 x 8192 38.8 -> 28.0, 224 x 13616 x 4096 23.0 -> 20.5,
    // 600 x 6144 x 4096 22.6 -> 19.7 against 14; with several rounds the two workgroups per CU of 14 overlap their tile
    // boundaries and win (2048 x 14336 x 4096: 105 against 124 us).
    // (Tried: workgroups starting at different places of K, against all of them asking for the same lines of every row
    // at a time -- no difference at K = 4096, 8192 and 14336.)
    {20, 128, 128, false, 2.230f, 2.657f, .548f, 0.f, .226f, .120f, .006f},
    // operands line by line into registers, K split over eight waves (gemm_packed_stream.hip).  Fitted to 675 shapes of M 17 ..
    // 16384, weights in the memory-side cache, after its loads became whole lines: on 500 others the choice is 0.5 % behind the
    // fastest configuration (14 % at worst), with the coefficients before 1.6 % (28 %).
    {64064, 64, 64, false, 1.579f, 1.873f, .225f, 0.f, .042f, .187f, .021f},
    {48064, 48, 64, false, 1.594f, 1.735f, .179f, 0.f, .035f, .209f, .039f},
    {48032, 48, 32, true, 1.462f, 1.272f, .259f, .128f, .012f, .403f, .059f},
    {32064, 32, 64, true, 1.335f, 1.672f, .289f, .153f, .023f, .293f, .060f},
    {32032, 32, 32, true, 1.795f, .826f, .197f, .097f, .005f, .389f, .057f},
    {32016, 32, 16, false, 2.145f, .414f, .055f, 0.f, 0.f, .545f, .055f},
};
constexpr GemmShape packed_shape(int64_t M, int64_t N, int64_t K, int64_t cus) { return {M, N, K, 256, .5f, cus}; }
constexpr const GemmConfig *packed_config(const GemmShape &s)
{
    // between the two large tiles the cheaper schedule of whole rounds (in outputs) decides, ties to the larger tile: with
    // many rounds of few stages that is right where the predictions are not (8192 x 14336 x 256: 70 against 75 us)
    const GemmConfig &small = kPackedConfigs[0], &large = kPackedConfigs[1];
    const bool larger = gemm_rounds(large, s) * large.bm <= gemm_rounds(small, s) * small.bm;
    return gemm_cheapest(kPackedConfigs, larger ? &large : &small, larger ? &small : &large, s);
}

template <int COUNT> constexpr bool coefficients_grow(const GemmConfig (&configs)[COUNT])
{
    for (const GemmConfig &c : configs) {
        if (c.fixed <= 0.f || c.per_round < 0.f || c.stage_tile < 0.f || c.out_mb < 0.f || c.weights_mb < 0.f) return false;
        if (c.stage_round <= 0.f || (c.pairs && (c.stage_lone <= 0.f || c.stage_lone > c.stage_round))) return false;
    }
    return true;
}
static_assert(coefficients_grow(kF6Configs) && coefficients_grow(kPackedConfigs), "a prediction may not fall where work is added");

// Whether the register kernel of the FP6 GEMM (tiles of 16 FM x 16 FN) fetches the 8-byte tails of two fragments at a time.  That
// takes L1 lookups away, and a few registers.  It gains where several rows of tiles read the same weights (240 shapes, M 17 .. 334: 1
// .. 5 % per tile, up to 12 %); with one row, or two of the wide tiles, memory bounds the launch (63 x 11040 x 2048, from HBM, 7.9 ->
// 8.5 us with pairs; 70 x 8048 x 8192 11.9 -> 12.4).  32 x 64 grows from 128 registers to 155, so one workgroup fits a CU instead of
// two: there only while every workgroup has a CU to itself (84 x 10464 x 2048, 492 of them on 256, 6.9 -> 8.1; 128 x 4096 x 14336, 256
// of them, 14.5 -> 14.2, weights from HBM 19.9 -> 18.6).
constexpr bool f6_pairs_tails(int64_t tiles_m, int64_t tiles_n, int fm, int fn, int64_t cus)
{
    return 2 * tiles_m > fn && (fm * fn != 8 || tiles_m * tiles_n <= cus);
}

// ---- tiles and workgroups (device code too: constexpr) ------------------------------------------------------------------
// Split of the tile grid over the 8 XCDs (each with its own L2): XCD x = v & 7 gets the rectangle
// (x % xcd_m, x / xcd_m) of an xcd_m x (8 / xcd_m) split and walks it m fastest.  Measured (FETCH_SIZE,
// M = 2048, K = 4096, int8 kernel): two halves in m by four blocks in n reads 112 MB through the fabric at
// N = 14336 where one run of tiles per XCD read 223 MB (half of X then stays in an XCD's 4 MB L2); it was
// also the fastest split at K = 14336.  Otherwise: the split whose rectangles need the fewest operand rows.
// A grid that does not divide into rectangles (kXcdRuns): bands of 8 rows of tiles, walked m fastest, cut into 8 runs of
// equal length, one per XCD: without it every XCD asks for nearly all of both operands (FP6, M 100 .. 6000, 72 ragged grids:
// 6.8 % faster on average; 762 x 24288 x 8192 143 -> 119 us, 390 x 7792 x 4096 18.4 -> 15.0, 5713 x 6512 x 4096 120 -> 105; packed
// nibbles, 74 grids: 3.2 %; 2871 x 9392 x 2048 62.5 -> 57.9).
// 0 = tile v is tile v of the grid, m fastest (by the knob, and for the 128 x 64 tiles of the FP6 kernel in place of runs).
constexpr int kXcdRuns = -1;
constexpr int choose_xcd_split(int tiles_m, int tiles_n, int BM, int BN)
{
    if (tiles_m % 2 == 0 && tiles_n % 4 == 0) return 2;
    int xcd_m = kXcdRuns;
    int64_t best = 0;
    for (int sm = 1; sm <= 8; sm *= 2) {
        if (tiles_m % sm != 0 || tiles_n % (8 / sm) != 0) continue;
        const int64_t rows = (int64_t)(tiles_m / sm) * BM + (int64_t)(tiles_n / (8 / sm)) * BN;
        if (xcd_m < 0 || rows < best) { xcd_m = sm; best = rows; }
    }
    return xcd_m;
}

// workgroups of a launch that holds `most` at a time (kXcdRuns: a multiple of 8, so that a workgroup's tiles stay in its XCD)
constexpr int64_t tile_workgroups(int64_t most, int64_t tiles, int xcd_m)
{
    if (xcd_m == kXcdRuns) tiles = (tiles + 7) / 8 * 8;
    return most < tiles ? most : tiles;
}

// Rows per tile of the FP6 kernel with two rows of waves: bm, or fewer where the rows of tiles, made equally high, leave whole
// fragments of 32 rows out (a multiple of 16 and more than bm / 2: the second row of waves has a fragment at least).
constexpr int f6_row_step(int64_t M, int bm)
{
    const int64_t tiles = (M + bm - 1) / bm, step = ((M + tiles - 1) / tiles + 15) / 16 * 16;
    return (step + 31) / 32 * 32 < bm && step > bm / 2 ? (int)step : bm;
}

// whether virtual workgroup v has a tile (if not, nor has v + any multiple of the grid); without divisions: it is asked between
// the last product and the stores of a tile
constexpr bool tile_exists(int v, int tiles_m, int tiles_n, int xcd_m)
{
    const int64_t total = (int64_t)tiles_m * tiles_n, x = v & 7;
    return xcd_m == kXcdRuns ? (x * total >> 3) + (v >> 3) < ((x + 1) * total >> 3) : v < total;
}

// its origin under that split
constexpr void tile_origin(int v, int tiles_m, int tiles_n, int xcd_m, int BM, int BN, int &m0, int &n0)
{
    int tm = 0, tn = 0;
    if (xcd_m > 0) {
        const int x = v & 7, l = v >> 3;
        const int rm = tiles_m / xcd_m, rn = tiles_n / (8 / xcd_m);      // rectangle size in tiles
        // walk: mw tiles in m fastest, then across the rectangle in n, then the next mw rows of tiles -- the ~32
        // tiles an XCD works on at a time then form a block of 8 x 4 tiles instead of a 32 x 1 column
        // (M = 16384, N = 4096, K = 4096 on the FP6 kernel: 148.6 -> 139.5 us)
        const int mw = (rm > 8 && rm % 8 == 0) ? 8 : rm;
        const int a = l % mw, b = (l / mw) % rn, c = l / (mw * rn);
        tm = (x % xcd_m) * rm + c * mw + a;
        tn = (x / xcd_m) * rn + b;
    } else if (xcd_m == kXcdRuns) {
        const int idx = (int)((int64_t)(v & 7) * tiles_m * tiles_n >> 3) + (v >> 3);
        const int band = idx / (8 * tiles_n), r = idx - band * 8 * tiles_n;
        const int h = tiles_m - 8 * band < 8 ? tiles_m - 8 * band : 8;
        tm = 8 * band + r % h;
        tn = r / h;
    } else {
        tm = v % tiles_m;
        tn = v / tiles_m;
    }
    m0 = tm * BM;
    n0 = tn * BN;
}

}  // namespace sr
