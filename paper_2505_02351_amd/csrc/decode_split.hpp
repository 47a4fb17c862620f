// How many units a decode launch over 8-bit caches makes of its tiles, and how they are taken: host code, nothing of HIP.
#pragma once
#include <stdint.h>

namespace optgqa {

// 8-bit caches, head_dim 128: the tiles (16 tokens of a segment) from which a launch's units are one to a SIMD, taken two tiles at a time;
// with fewer, two to a SIMD, tile by tile.  0: never, whatever the lengths, for launches whose tiles under the caller's bound are fewer than
// kPairUnitTiles to a SIMD.  The host asks by the bound which kernel to launch, and that kernel compares the tiles that there are.
//
// A tile is half a 2-byte cache's bytes, its chain of widening, scores, softmax, V through LDS and output products as long.  Tile by tile
// the chain sets one wave's pace, and two waves to a SIMD, which share it, stream less evenly than one (the older runs ahead).  Two tiles' chains
// side by side keep one wave busy, with as many bytes on their way as a 2-byte cache's.  But a segment's start and end are a chain that
// nothing of the same wave hides: where a unit has several segments' pieces, a second wave does, until they are long.
// Steps, us, tile by tile | in pairs if always | as chosen (bf16, slopes, in graphs, several sets of caches in turn):
//   64 sequences, 32 / 4 heads (256 segments to 1 024 SIMDs): of 50-400 15.6 | 14.2 | 14.5, of 255-2 047 26.0 | 24.5 | 25.5,
//       of 1 023-8 191 64.1 | 59.9 | 60.4
//   64, 32 / 8 (512): of 15-127 13.3 | 15.6 | 13.3, of 127-1 023 24.1 | 24.9 | 24.1, of 375-3 000 49.0 | 46.7 | 47.3,
//       of 1 023-8 191 109.9 | 107.4 | 107.4
//   100, 32 / 8 (800): of 127-1 023 31.5 | 33.8 | 31.4, of 255-2 047 49.4 | 49.4 | 49.6, of 1 023-8 191 153.0 | 148.6 | 148.6
//   200, 32 / 8 (1 600): of 15-127 21.9 | 33.2 | 21.5, of 63-511 34.4 | 42.2 | 34.3, of 255-2 047 87.1 | 91.6 | 87.1, of 1 023-8 191 320 | 310 | 310
//   8, 32 / 8 (64): of 50-400 11.0 | 12.7 | 11.2, of 511-4 095 16.4 | 16.5 | 16.4, of 1 023-8 191 24.1 | 23.2 | 23.8
// (the choice itself, twice as many waves of which half end at once, costs 0.2 to 0.5 us).  head_dim 64, 64 of 1 023-8 191: 39.0 and 44.9, never.
constexpr int kPairUnitTiles = 32;

// segments: sequences x KV heads x head chunks; rows: sequences x heads; units: SIMDs (four to a CU).  Few rows are combined by
// groups of threads that read many pieces side by side, so that fewer units save little there.
inline int decode_pairs_from(int64_t segments, int64_t rows, int max_context_len, int cus)
{
    const int64_t units = 4ll * cus;
    if (segments * ((max_context_len + 15ll) / 16) < kPairUnitTiles * units) return 0;
    const int64_t tiles = (rows <= units ? 18 : 2) * units + 160 * (segments > units / 4 ? segments - units / 4 : 0);
    return tiles < 0x7fffffff ? (int)tiles : 0x7fffffff;
}

}  // namespace optgqa
