// Which workgroup shape a prefill launch takes: host code, nothing of HIP.
#pragma once
#include <stdint.h>

namespace optgqa {

// Shapes of a prefill workgroup (see prefill_kernels.hpp): 128 rows, 256 rows, or 128 rows whose keys are
// shared out between two groups of four waves.
enum class PrefillShape { k4Waves, k8Waves, k8WavesTwoGroups };

// Query tiles of a sequence of max_q_len new tokens in workgroups of 32 * waves rows.
inline int64_t prefill_q_tiles(int waves, int heads_pow2_shift, int max_q_len)
{
    const int tokens = (waves * 32) >> heads_pow2_shift;
    return ((int64_t)max_q_len + tokens - 1) / tokens;
}

// units8: (sequence, KV head, head chunk) triples rounded up to 8s; max_q_len: the caller's bound on the new tokens.
// In order (GPU time of passes in us; bf16, 32 / 8 heads, head_dim 128, slopes, where nothing else is said; see also
// prefill_kernels.hpp):
//   a window              -> 128 rows, which span few keys.  8 chunks of 512, no slopes, with the cache write:
//                              window              64     512   1 024   2 048   4 096
//                              256 rows          36.2    75.4   117.8   204.5   220.6
//                              128 rows          30.7    70.1   116.3   211.5   235.9
//   128-row workgroups fill the CUs at most once
//                         -> two key groups, which halve the longest walk (a workgroup whose walk is short uses one,
//                            kPfTwoGroupTiles):
//                              workgroups           160     256     256     512     512     512
//                                        634 > 1 723 e4m3  1 x 1 024  2 x 512 > 2 048  2 x 1 024  2 x 1 024 > 2 048  4 x 512 > 2 048
//                              two groups          55.4    25.8    57.2    35.6    92.9    80.9
//                              128 rows            66.8    29.9    70.6    37.4    92.4    78.2
//   256-row workgroups would not fill them twice
//                         -> 128 rows, two workgroups to a CU.  Chunks behind 2 048:
//                              256-row workgroups   256     384     448     512     512, no slopes
//                                               4 x 512  6 x 512 8 x 448 8 x 512  8 x 512
//                              256 rows            92.7    99.3    98.7   111.7   218.1
//                              128 rows            78.2    99.5   107.1   122.2   235.9
//   whole prompts, not five times
//                         -> 128 rows: the walks are short against what a workgroup costs before and behind its
//                            walk, which two resident workgroups overlap.  8 prompts:
//                              tokens, and workgroups  768  1 024  1 280   1 280, no slopes   1 280, head_dim 64   1 536   2 560
//                              256 rows               69.1  105.2  141.3   186.6               97.8                190.1   385.1
//                              128 rows               65.9  100.7  134.2   177.5               81.6                184.2   395.6
//   else                  -> 256 rows: half the loads and LDS stores per row.
// The lines date from a longer start of a workgroup; with today's, windows of 2 048 and chunks that fill the CUs 1.75 times are
// faster with 256 rows, and whole prompts with 128 up to six times (none of it tried over the ranges that a line serves).
// What is counted are workgroups under the caller's bound: most of them may find no tokens, and then the launch is smaller
// than it looks.  So prompts do not take 256 rows for a large bound alone, though prompts of 2 048 and more that are that
// long gain by it (256 and 128 rows: 4 of 2 560 182.5 and 190.6, 2 of 2 560 108.9 and 110.4; but under bounds of that size
// 4 of 768 40.6 and 37.2, 5 of 1 024 65.4 and 60.9, 2 of 173 12.9 and 10.4, one of 2 048 under 8 192 74.3 and 63.2).
inline PrefillShape prefill_shape(int64_t units8, int heads_pow2_shift, int max_q_len, bool windowed, bool whole_prompts, int cus)
{
    const int64_t blocks8 = units8 * prefill_q_tiles(8, heads_pow2_shift, max_q_len);
    const int64_t blocks4 = units8 * prefill_q_tiles(4, heads_pow2_shift, max_q_len);
    if (windowed) return PrefillShape::k4Waves;
    if (blocks4 <= cus) return PrefillShape::k8WavesTwoGroups;
    if (blocks8 < 2 * cus || (whole_prompts && blocks8 <= 5 * cus)) return PrefillShape::k4Waves;
    return PrefillShape::k8Waves;
}

}  // namespace optgqa
