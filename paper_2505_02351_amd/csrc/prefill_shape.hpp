// Which workgroup shape a prefill launch takes, and which block numbers a wave holds: nothing of HIP.
#pragma once
#include <stdint.h>

namespace optgqa {

// Lane l of a wave holds the number of its sequence's block `first` - l: whether one holds that of `block` (lane first - block).
// A walk goes down the blocks, but where it is started anew after loads were asked for further on, it may go up.
constexpr bool held_blocks_reach(int first, int block) { return (uint32_t)first - (uint32_t)block < 64u; }

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
// For tiles that pass through registers (8-bit caches), with which all its figures were measured; for those that do not it is
// prefill_shape_direct's starting point.  In order (GPU time of passes in us; bf16, 32 / 8 heads, head_dim 128, slopes, where nothing else is said; see also
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
// What is counted are workgroups under the caller's bound: most of them may find no tokens, and then the launch is smaller
// than it looks.
inline PrefillShape prefill_shape(int64_t units8, int heads_pow2_shift, int max_q_len, bool windowed, bool whole_prompts, int cus)
{
    const int64_t blocks8 = units8 * prefill_q_tiles(8, heads_pow2_shift, max_q_len);
    const int64_t blocks4 = units8 * prefill_q_tiles(4, heads_pow2_shift, max_q_len);
    if (windowed) return PrefillShape::k4Waves;
    if (blocks4 <= cus) return PrefillShape::k8WavesTwoGroups;
    if (blocks8 < 2 * cus || (whole_prompts && blocks8 <= 5 * cus)) return PrefillShape::k4Waves;
    return PrefillShape::k8Waves;
}

// The shape where tiles go to LDS directly (2-byte caches and inputs): a tile's loads cost 128 rows little more than 256, so two
// workgroups of 128 rows, which hide each other's start, end and barriers, win over more of the range.  slopes: given.  (As above; 256 rows, and
// 128; what the general rule gives goes for windows and two key groups.)
//   head_dim 64           -> 128 rows, always:
//                                        8 x 2 560  16 x 2 560, no slopes  8 x 512 > 2 048  16 x 512 > 2 048  8 x 512 > 2 048, no slopes
//                              256 rows     233.9        812.7                  69.5             134.5              132.0
//                              128 rows     188.3        697.7                  67.1             123.5              127.1
//   no slopes             -> 128 rows: nothing is skipped, and all steps of a workgroup are alike.  24 ragged chunks 231.8 and 213.4, 8 prompts
//                            of 2 560 601 and 585, 16 of them 1 210 and 1 195, chunks of 512 behind 2 048: 6 182.9 and 159.8, 7 189.4 and
//                            193.1, 8 209.9 and 208.7.
//   256-row workgroups would not fill the CUs 1.75 times
//                         -> 128 rows.  Chunks of 512 behind 2 048:
//                              256-row workgroups      256     384     448     512    1 024
//                              256 rows               90.6    94.4   100.6   105.8    213.7
//                              128 rows               72.3    92.5   105.5   114.1    229.0
//   whole prompts whose bound is at most 3 072 tokens, or that 256-row workgroups fill not five times
//                         -> 128 rows; in a longer walk the loads that 256 rows save weigh more.  8 prompts:
//                              tokens                 1 024   1 536   2 560   2 560, 16 prompts   4 096   2 560, fp16
//                              256 rows                95.6   183.5   375.0        725.1           705.6      345.8
//                              128 rows                88.6   165.7   355.5        723.2           732.3      321.3
//   else                  -> 256 rows.
inline PrefillShape prefill_shape_direct(int64_t units8, int heads_pow2_shift, int max_q_len, int head_dim, bool slopes, bool windowed,
                                         bool whole_prompts, int cus)
{
    const PrefillShape any = prefill_shape(units8, heads_pow2_shift, max_q_len, windowed, whole_prompts, cus);
    if (windowed || any == PrefillShape::k8WavesTwoGroups) return any;
    const int64_t blocks8 = units8 * prefill_q_tiles(8, heads_pow2_shift, max_q_len);
    if (head_dim == 64 || !slopes || 4 * blocks8 < 7 * cus) return PrefillShape::k4Waves;
    if (whole_prompts && (blocks8 <= 5 * cus || max_q_len <= 3072)) return PrefillShape::k4Waves;
    return PrefillShape::k8Waves;
}

}  // namespace optgqa
