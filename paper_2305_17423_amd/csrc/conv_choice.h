// Which kernel a convolution outside the bf16 matrix path and a fresh GroupNorm of a map take: plain C++, so that a host program can ask for the form of any
// size.  Internal.
#pragma once

namespace fise {

// ---- conv.hip, fp32: the edge of the tiles that eight waves share K of, 0: the staged kernel.
// Up to one 32 x 32 tile per CU it is the faster one at every size measured (8 - 256 tiles; us here / staged at 256): 3x3 of 16
// channels 5.3 / 8.8, 64 9.2 / 20.1, 320 27 / 84, 1280 101 / 324; 1x1 of 16 4.3 / 4.4, 64 5.2 / 5.7, 1280 15 / 39.  A second tile per CU
// costs a second round: at 320 tiles 1x1 of 64 channels 7.3 / 5.8, of 128 7.7 / 7.5, though 3x3 of 64 still 15 / 20.
// Of its two tiles 16 x 16 while there are at most two for each CU (detection and convolution alone, us, 32 x 32 and 16 x 16): 40 tiles of 64 channels
// 29.1, 26.4; 256 of 128 channels 33.5, 28.4; 512 of 64 29.2, 27.9; 960 of 64 29.4, 32.1.
// Pixel numbers of the output have 32 bits.
inline int conv_f32_edge(int rows, int Cout, long long pixels) {
    auto tiles = [&](int e) { return (long long)((rows + e - 1) / e) * ((Cout + e - 1) / e); };
    if (tiles(32) > 256 || pixels >= 1ll << 31) return 0;
    return tiles(16) <= 512 ? 16 : 32;
}

// ---- conv.hip, four columns behind a GroupNorm: whether conv_out_kernel takes them.  Its patch of 640 channels is 47 of the 64 KB of LDS that a launch has without asking
// (896 do not fit); workgroups of 4 x 4 pixels; their numbers have 24 bits.
constexpr int CO_MAX_C = 640;
struct ConvOut { int C0, C1, Cout, ksize, stride, tile, tile_w, n_active; bool upsample, groupnorm, adds; };      // adds: time projection, residual or normalised copies
inline bool conv_out_takes(const ConvOut& a) {
    return a.groupnorm && a.C1 == 0 && a.C0 <= CO_MAX_C && a.Cout == 4 && a.ksize == 3 && a.stride == 1 && !a.upsample && !a.adds && a.tile % 4 == 0 && a.tile_w == a.tile &&
           (long long)a.n_active * (a.tile / 4) * (a.tile / 4) < 1 << 24;
}

// ---- norm.hip, fresh statistics and activation of a map of which every pixel is active: one launch (gn_map_kernel) or two.
constexpr int GM_THREADS = 512, GM_MAX_J = 8, GM_MAX_GROUPS = GM_THREADS / 64;      // a wave finishes a group
// Slab of a workgroup: the fewest whole groups whose channels are a multiple of 8.
struct GnSlab { int groups, pieces; };
inline GnSlab gn_slab(int C, int G) {
    const int cpg = C / G, unit = cpg % 8 == 0 ? 1 : cpg % 4 == 0 ? 2 : cpg % 2 == 0 ? 4 : 8;
    if (cpg < 8 || G % unit) return {0, 0};
    return {unit, unit * cpg / 8};
}
// Pieces a lane of gn_map_kernel holds, 0: two launches.  Up to eight: 32 workgroups of eight 9.5 us (two launches 10.4), of twelve 10.6 (10.1) with 512 lanes
// as with 1024, 64 of twelve 12.6 (12).  Fewer than 32 workgroups were not measured.  Channels: what the statistics' launch takes.
inline int gn_map_values(const GnSlab& s, int B, int HW, int C, int G) {
    if (!s.groups || C > 64 * 1024 / 16 || s.pieces > GM_THREADS || (long long)B * (G / s.groups) < 32) return 0;
    const int lanes = GM_THREADS / s.pieces, n = (HW + lanes - 1) / lanes;
    return n <= GM_MAX_J ? n : 0;
}

}  // namespace fise
