// Which tile and K split a launch of wave_gemm.hip takes, which row tile one of linear_wide.hip, which tile and column units one of norm_gemm.hip: plain C++,
// so that a host program can ask for the form of any size.  Internal.
#pragma once
#include <algorithm>
#include <cstddef>

namespace fise {

// Scratch of the launcher: the parked partial sums of split-K launches, then the arrival counters.
constexpr int IGEMM_COUNTERS = 4096;     // arrival counters of split output tiles (zeroed once per call, left at zero by every launch)
constexpr size_t IGEMM_PARTIAL_BYTES = (32u << 20) - IGEMM_COUNTERS * sizeof(int);

// Tile and K split of a launch: the cheapest of the combinations under times measured per part of a launch (us, from time
// stamps inside the kernel and kernel traces over the shapes of steps and dense builds).
//  - PRIVATE, a ring per wave, 256 workgroups at once.  `fixed`: start, row positions, first loads, sum over the waves,
//    epilogue, and the gap to the launch before.  `iter`: four K steps, one per wave (operands at the 71 - 88 GB/s a CU gets with all busy).
//  - SHARED, 64 x 64 on one ring of 48 KB: every wave multiplies a 16-deep slice of each K step over the whole tile, so a
//    staged byte is read once, and three workgroups per CU hide each other's start and epilogue, which many tiles of
//    a short K consist of: `tile` + `iter` per K step of a tile and CU.  4096 x 320 x 2880, stride 2, 24 us (PRIVATE 28), 8192 x 640 x 5760,
//    upsampling, 76 (93); with GEGLU 1376 x 5120 x 640 39 -> 26 us.  Beyond ~96 K steps (`iter_long`) the workgroups of an XCD drift apart and fall
//    out of its L2.
//  - BLOCK, 64 x 160 on one ring of 112 KB: 1/46 of an operand row per product instead of 1/32, one workgroup per CU and a
//    long epilogue (ten pieces per thread): 4096 x 640 x 5760, stride 2, 44 us (SHARED 74), 2048 x 1280 x 11520, stride 2, 87 (139).  Widths of a
//    320-channel UNet are multiples of 160: no columns to spare.
// A K split over workgroups adds parking, counting and re-reading the tiles (`park`, `park_s` per split).
// kShapes serves what the forms below do not take: stride 2, upsampling, tiles of edge 1, 1x1 over maps, compact rows.  Its constants come from time
// stamps and from 3x3 convolutions that kPatchShapes has now.  Held against every tile and split on 173 launches of its own (widths
// 320 / 640 / 1280, K up to 23040, 2 to 8192 rows, cold weights), the choice is 4 % from the best on average over stride 2, 7 % over upsampling, 3 % over
// edge 1 and 1 % over compact rows.  It is furthest off at 90 - 180 K steps and 80 - 320 tiles: 1376 x 1280 x 11520, upsampling, 80 us (BLOCK; SHARED
// 61); 512 x 1280 x 11520, upsampling, 41 (BLOCK in four; SHARED in three 34); 2048 x 640 x 5760, stride 2, 43 (SHARED; BLOCK in two 32).  The same
// form is up to 1.7 times as slow under stride 2 as under upsampling (8192 x 640 x 5760 on SHARED 134 us and 76), which one `iter` does not tell apart.
//  - PATCHES, 3x3 convolutions of stride 1 over square tiles of edge 2, 4 or 8, `iter` per chunk of 64 channels (times `small` at edge 2,
//    whose patches are four times the tile): the other forms bring a pixel into LDS once per tap, this one brings the tiles' patches
//    in once, 1/5 (edge 8) to 1/2 (edge 2) of the bytes.  1376 x 640 x 5760: 23.3 -> 18.8 us, 1536 x 320 x 8640 21.7 -> 17.2, 344 x
//    1280 x 11520 29.5 -> 23.  It loses where few rows leave a launch its fixed cost (64 rows), its set-up being longer.
// These launches have a table of their own, kPatchShapes: fitted to every form and split of 127 convolutions (320 / 640 / 1280 wide, 4 to 18432 rows, tiles
// of edge 2 to 8, cold weights), where the choice is 0.6 % from the best on average, at worst 9 %, and 10 % faster than without PATCHES.
//  - WIDE, the same over 64 or 128 rows x 80 columns (conv_patch.hip), edge 4 (64 rows) or 8: fewest bytes per product, one workgroup per CU, for
// launches that give most CUs one of its tiles.  8192 x 320 x 2880 29 -> 21.5 us, x 8640 67 -> 47; 4096 x 320 x 5760 37 -> 22.7; 2048 x 640 x 5760
// 35 -> 24.3, x 17280 76 -> 58; not for 2432 x 320 x 2880 (152 tiles: 14 against 12.7) or 4608 x 640 x 5760 (576: 62 against 54).
enum { PRIVATE = 0, SHARED_RING = 1, BLOCK = 2, PATCHES = 3, WIDE = 4 };
struct TileShape { int kind, tm, tn; double fixed, tile, iter, iter_long, park, park_s, small; };
inline constexpr TileShape kShapes[] = {
    {PRIVATE, 1, 1, 4.3, 0.0, 0.39, 0.39, 2.0, 0.15, 1}, {PRIVATE, 1, 2, 4.8, 0.0, 0.56, 0.56, 2.3, 0.3, 1}, {PRIVATE, 2, 2, 5.8, 0.0, 0.92, 0.92, 3.2, 0.6, 1},
    {SHARED_RING, 2, 2, 5.2, 1.2, 0.235, 0.32, 3.2, 0.6, 1}, {BLOCK, 2, 5, 13.0, 0.0, 0.4, 0.4, 4.0, 1.5, 1}};
inline constexpr TileShape kPatchShapes[] = {
    {PRIVATE, 1, 1, 4.4, 0.0, 0.25, 0.39, 2.0, 0.15, 1}, {PRIVATE, 1, 2, 4.8, 0.0, 0.56, 0.56, 2.5, 0.3, 1}, {PRIVATE, 2, 2, 5.8, 0.0, 0.92, 0.92, 3.2, 0.6, 1},
    {SHARED_RING, 2, 2, 5.2, 1.2, 0.25, 0.32, 3.2, 0.6, 1}, {BLOCK, 2, 5, 11.8, 0.0, 0.4, 0.365, 4.0, 1.5, 1},
    {PATCHES, 1, 1, 4.9, 0.0, 0.52, 0.6, 4.0, 0.15, 1}, {PATCHES, 2, 1, 6.6, 0.0, 0.69, 0.69, 3.1, 0.3, 1.1}, {PATCHES, 2, 2, 7.0, 0.0, 1.05, 1.0, 4.3, 0.6, 1.2},
    {WIDE, 2, 0, 6.6, 0.0, 1.68, 1.68, 0.0, 0.0, 1}, {WIDE, 4, 0, 8.9, 0.0, 2.5, 2.5, 0.0, 0.0, 1}};
constexpr double PATCH_SIDE = 0.25;          // a K step of the side product behind the chunks

// What the choice depends on.  K2: channels of the side product; tile: edge (rows of compact buffers: any); patches: 3x3 over strips that have a
// patch form; one_map: pixels of maps into one bf16 map, with a map as residual if any.
struct GemmShape { int rows, N, K, K2, tile; bool geglu, patches, one_map; };
struct TileChoice { int kind, tm, tn, splits; };
// partial_bytes: scratch for parked sums (0: no K split).
inline TileChoice choose_tile(const GemmShape& a, size_t partial_bytes) {
    auto up = [](int n, int d) { return (n + d - 1) / d; };
    const int ncols = a.geglu ? 2 * a.N : a.N, nsteps = (a.K + a.K2) / 64;
    TileChoice c{PRIVATE, 1, 1, 1}; double best = 1e30;
    const int max_s = partial_bytes ? 8 : 1;
    const TileShape* const table = a.patches ? kPatchShapes : kShapes;
    for (int i = 0; i < (int)(a.patches ? sizeof kPatchShapes : sizeof kShapes) / (int)sizeof(TileShape); ++i) {
        const TileShape& sh = table[i];
        if (a.geglu && sh.tn == 1) continue;
        if (sh.kind == BLOCK && (!a.one_map || a.N % 160)) continue;
        if (sh.kind == PATCHES && sh.tm == 1 && a.tile == 2) continue;      // never the cheapest
        if (sh.kind == WIDE && (a.N % 80 || !(a.tile == 8 || (a.tile == 4 && sh.tm == 2)))) continue;
        const bool chunks = sh.kind == PATCHES || sh.kind == WIDE;
        const int gx = up(a.rows, 32 * sh.tm), gy = sh.kind == WIDE ? a.N / 80 : up(ncols, 32 * sh.tn), pieces = chunks ? a.K / 576 : nsteps;
        for (int s = 1; s <= max_s; ++s) {
            const int per = up(pieces, s);
            if (s > 1 && (sh.kind == WIDE || (sh.kind != PATCHES && per < 4) || up(pieces, per) != s)) continue;
            if (s > 1 && ((long long)gx * gy > IGEMM_COUNTERS || (size_t)gx * gy * s * 32 * sh.tm * 32 * sh.tn * 4 > partial_bytes)) break;
            const long long n = (long long)gx * gy * s;
            const double iter = (nsteps > 96 ? sh.iter_long : sh.iter) * (a.tile == 2 ? sh.small : 1);
            double t = s > 1 ? sh.park + sh.park_s * s : 0.0;
            if (sh.kind == SHARED_RING) t += sh.fixed + std::max(1.0, n / 256.0) * (sh.tile + per * iter);
            else t += (double)((n + 255) / 256) * (sh.fixed + (sh.kind == PRIVATE ? up(per, 4) : per) * iter + (chunks ? up(a.K2 / 64, s) * PATCH_SIDE * (sh.kind == WIDE ? 0.5 * sh.tm : 1.0) : 0.0));
            if (t < best) { best = t; c = {sh.kind, sh.tm, sh.tn, s}; }
        }
    }
    return c;
}

// linear_wide.hip: row tiles of 32 of a launch, 0: igemm.hip's tiles.  One tile for each CU at most: 64 rows while that suffices, else 128 (several rounds of them
// fall behind 64 x 128 tiles, of which a CU holds two: 9216 x 320 x 320 11.7 us there, 12.0 and 14.4 here; 9216 x 640 x 2560 57, 63 and 67).
// Fewer than 2048 rows belong to wave_gemm.hip, which splits K over more waves.  Before and now, us: 2048 x 320 x 1280 14.0, 8.3; 2048 x 640 x 640
// 9.9, 6.9; x 2560 23.2, 13.7; 4096 x 320 x 320 8.0, 5.5; 5504 x 320 x 1280 19.0, 13.4; 8192 x 320 x 320 11.2, 8.9; x 1280 20.7, 14.5; 2048 x 1280 x 5120
// 64, 42.
inline int linear_tile(int rows, int N) {
    const long long columns = N / 80;
    if (rows < 2048 || (rows + 127) / 128 * columns > 256) return 0;
    return (rows + 63) / 64 * columns <= 256 ? 2 : 4;
}

// ---- rows_group.hip: row tiles of 32 a workgroup takes, 0: the tiles of wave_gemm.hip.  One workgroup runs per CU; a round costs its start and epilogue (as
// much as the operands of 290 rows of stages) and the rows of both operands that it loads.  The smaller tiles of wave_gemm.hip fill the chip where
// there are few columns: their time goes with the number of columns, a round's does not (24960 columns, 154 rows: 24.0 and 15.5 us).  With several rounds the two
// are held against each other, us at 24960 columns of 768 channels: 6.5 and 3.7 + 1.5 rt a round; 12.7 and 3.83 for every 64 rows, where a batch element's rows are a
// multiple of four (`fours`: transposed columns go out four rows at a time), else 15 and 4.75.  There and here: 240 rows 28.2, 28.9, 264 30.1, 28.6, 448
// 38.6, 36.2, 512 43.1, 48.9, 576 46.5, 49.5; no fours 226 33.7, 29.0, 520 57.1, 49.1.
constexpr int GROUP_UNITS = 7;               // units of 16 columns of a workgroup
inline int group_tile(int rows, int cols, bool fours) {
    constexpr int kTiles[] = {1, 2, 3, 5, 7};
    const long long groups = (cols / 16 + GROUP_UNITS - 1) / GROUP_UNITS;
    int best = 0; double least = 1e30; long long rounds = 0;
    for (const int rt : kTiles) {
        const long long n = ((rows + 32 * rt - 1) / (32 * rt) * groups + 255) / 256;
        const double t = (double)n * (290 + 32 * rt + 16 * GROUP_UNITS);
        if (t < least) { least = t; best = rt; rounds = n; }
    }
    const double here = 6.5 + rounds * (3.7 + 1.5 * best), there = (fours ? 12.7 + 3.83 * ((rows + 63) / 64) : 15 + 4.75 * ((rows + 63) / 64)) * (cols / 24960.0);
    return groups >= 160 && (rounds == 1 || here <= there) ? best : 0;
}

// ---- norm_gemm.hip
constexpr int NG_WAVES = 8, NG_LDS_MAX = 160 * 1024, NG_BIAS = 5120;      // bytes of bias of a workgroup: 80 units of 32 columns

// Logarithm of the waves that share a unit: all there are, where their sums find room in the place of the rows (320 channels of 32 columns: not).  1280 channels,
// 24 rows: one product 8.1 -> 7.0 us, queries, keys and values 10.1 -> 8.5; 640 channels 384 rows 7.5 -> 7.2.
inline int waves_per_unit(int KM, int CT, int per) {
    int ks = 0;
    if (CT * 512 <= 640 * KM + (KM == 1 ? 0 : 128))
        while ((per << (ks + 1)) <= NG_WAVES && (2 << ks) <= 5 * KM) ++ks;
    return ks;
}

// Rows (16 rt) and columns (16 ct) of a workgroup's tile per width, stages of the weights in LDS.
#define FISE_NORM_TILES(T) /* K, GEGLU, rt, ct, stages */                                                                        \
    T(320, 1, 4, 2, 2) T(320, 1, 2, 2, 3) T(640, 1, 4, 2, 2) T(640, 1, 2, 2, 3) T(1280, 1, 2, 2, 2) T(1280, 1, 1, 2, 3)           \
    T(320, 0, 4, 2, 3) T(320, 0, 2, 1, 4) T(640, 0, 2, 2, 3) T(640, 0, 2, 1, 4) T(1280, 0, 2, 2, 2) T(1280, 0, 2, 1, 4) T(1280, 0, 1, 1, 4)
struct NormTile { int K, geglu, rt, ct, nd; };
#define FISE_NORM_TILE(K, GEGLU, RT, CT, ND) {K, GEGLU, RT, CT, ND},
inline constexpr NormTile kNormTiles[] = {FISE_NORM_TILES(FISE_NORM_TILE)};
#undef FISE_NORM_TILE

struct NormShape { int B, Ma, K, N; bool geglu, gn; };     // gn: a GroupNorm's (scale, shift) table in LDS
struct NormChoice { int tile, per; };                      // in kNormTiles (-1: none), column units of a workgroup
// The row tile and column units per workgroup of a launch: the cheapest under times (us) fitted to 800 combinations of tile and split over the
// products of 320 / 640 / 1280 channels with 16 to 8192 rows and cold weights, where the choice is 0.6 % from the best on average, at worst
// 10 %.  One workgroup runs per CU; a round of 256 pays for its rows (16 rows of 320 channels 0.66), for the LDS traffic of its units
// (2 RT + 4 CT KB a wave and stage of 64 channels) and for the stages a wave goes through; what all workgroups read of the weights comes on top.
inline NormChoice choose_norm_tile(const NormShape& a) {
    constexpr int kPer[] = {1, 2, 3, 4, 6, 8, 10, 12, 16, 20, 24, 32, 40, 64, 80};
    static_assert(kPer[14] * 32 * 2 <= NG_BIAS, "bias of a workgroup");
    auto up = [](int n, int d) { return (n + d - 1) / d; };
    const int rows = a.B * a.Ma, NK = a.K / 64, KM = a.K / 320;
    NormChoice c{-1, 1}; double best = 1e30;
    for (int i = 0; i < (int)(sizeof kNormTiles / sizeof(NormTile)); ++i) {
        const NormTile& t = kNormTiles[i];
        if (t.K != a.K || t.geglu != (int)a.geglu) continue;
        // the table holds two batch elements, and the smallest row tile is 32 (16 at 1280 channels)
        if (a.gn && a.B > 1 && a.Ma < 16 * t.rt) continue;
        if (a.gn && 16 * t.rt * (640 * KM + 136) + NG_WAVES * t.nd * t.ct * 2048 + NG_BIAS + 2 * a.K * 8 > NG_LDS_MAX) continue;
        const int units = a.N / (a.geglu ? 16 : 16 * t.ct), gx = up(rows, 16 * t.rt);
        for (const int per : kPer) {
            if (per > units) break;
            const long long wgs = (long long)gx * up(units, per);
            const int ks = waves_per_unit(KM, t.ct, per), stages = ks ? (NK + (1 << ks) - 1) >> ks : up(per, NG_WAVES) * NK;
            const double us = 1.8 + (double)((wgs + 255) / 256) * (2.0 + 0.66 * t.rt * KM + 0.0031 * per * NK * (2 * t.rt + 4 * t.ct) + 0.026 * stages + (ks ? 0.26 : 0.0)) +
                              0.024e-3 * wgs * per * NK * t.ct + 0.12 * NK * (t.ct - 1) / (1 << ks);
            if (us < best) { best = us; c = {i, per}; }
        }
    }
    return c;
}

}  // namespace fise
