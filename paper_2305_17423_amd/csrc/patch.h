// Geometry of the patches behind the BM rows of a workgroup (3x3, stride 1, square tiles of edge T): strips of H x T pixels with their
// one-pixel ring, in LDS as rows of 64 channels (128 bytes).  Internal.
#pragma once
#include "common.h"

namespace fise {

template <int BM, int T> struct Patch {
    static constexpr int H = BM / T < T ? BM / T : T, PIX = (H + 2) * (T + 2), STRIPS = BM / (H * T);
    static constexpr int SLOTS = (STRIPS * PIX + 31) / 32;      // 16-byte loads per lane and chunk of 64 channels
    static constexpr int BYTES = SLOTS * 32 * 128;
    // Segment of 16 bytes that slot 0 of patch row p holds.  The LDS serves sixteen lanes at once (0-3, 12-15, 20-23, 24-27 and so
    // on); under every tap their sixteen pixels lie in different (row parity, segment) pairs.
    static __device__ __forceinline__ int swizzle(int p) {
        const int strip = p / PIX, q = p % PIX;
        return (q % (T + 2) / 2 + T / 2 * (q / (T + 2)) + T * T / 2 * strip) & 7;
    }
};

}  // namespace fise
