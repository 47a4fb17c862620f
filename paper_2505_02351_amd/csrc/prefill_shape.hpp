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
// For tiles that pass through registers (8-bit caches: chunks only), with which all its figures were measured, e4m3 or before 2-byte tiles went to
// LDS directly.  In order (GPU time of passes in us; bf16, 32 / 8 heads, head_dim 128, slopes, where nothing else is said; see also
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
//   else                  -> 256 rows: half the loads and LDS stores per row.
// What is counted are workgroups under the caller's bound: most of them may find no tokens, and then the launch is smaller
// than it looks.
inline PrefillShape prefill_shape(int64_t units8, int heads_pow2_shift, int max_q_len, bool windowed, int cus)
{
    const int64_t blocks8 = units8 * prefill_q_tiles(8, heads_pow2_shift, max_q_len);
    const int64_t blocks4 = units8 * prefill_q_tiles(4, heads_pow2_shift, max_q_len);
    if (windowed) return PrefillShape::k4Waves;
    if (blocks4 <= cus) return PrefillShape::k8WavesTwoGroups;
    if (blocks8 < 2 * cus) return PrefillShape::k4Waves;
    return PrefillShape::k8Waves;
}

// Bytes of K and V rows that a launch reads, under the caller's bounds, that are more than the last-level cache keeps (256 MB).
constexpr int64_t kPrefillFarKeys = 320000000;

// The shape where tiles go to LDS directly (2-byte caches and inputs): a tile's loads cost 128 rows little more than 256, so two
// workgroups of 128 rows, which hide each other's start, end and barriers, win over more of the range.  slopes: given.  key_bytes: of K and V
// rows.  (As above; 256 rows, and 128; what the general rule gives goes for windows and two key groups.)
//   head_dim 64           -> 128 rows, always:
//                                        8 x 2 560  16 x 2 560, no slopes  8 x 512 > 2 048  16 x 512 > 2 048  8 x 512 > 2 048, no slopes
//                              256 rows     233.9        812.7                  69.5             134.5              132.0
//                              128 rows     188.3        697.7                  67.1             123.5              127.1
//   256-row workgroups would not fill the CUs twice; with slopes and two of them or more to a unit, not 1.75 times
//                         -> 128 rows.  Chunks behind 2 048, 1 000 and 1 000, heads 32 / 8, 32 / 8 and 16 / 16:
//                              256-row workgroups   256   384   448   512  1 024      464 (29 x 125)      480 (30 x 2: one to a unit)
//                              256 rows            90.6  94.4 100.6 105.8  213.7          90.1                   67.9
//                              128 rows            72.3  92.5 105.5 114.1  229.0          90.3                   51.1
//   no slopes             -> 128 rows: nothing is skipped, and all steps of a workgroup are alike (24 ragged chunks 231.8 and 213.4, 40 of 125 behind 1 000
//                            163.2 and 149.1), but 256 where the keys are more than the last-level cache keeps - equal chunks' tiles of rows start together, one
//                            sequence's far apart, and 128 read memory twice as often - or chunks are long (the bound stands for the length):
//                              16 / 16 heads       100 x 131 > 1 000 (927 MB)  40 x 1 021 > 1 000 (662)  64 prompts of 1 523 (399)  16 x 1 021 > 1 000 (265)
//                              256 rows                   340.1                     926.4                  1 271                     364.7
//                              128 rows                   430.4                   1 058                    1 505                     352.1
//                              32 / 8, chunks      16 x 509 > 300   5 x 1 604 > 2 097, fp16   40 x 1 500 > 300   8 x 2 560 > 300   8 x 4 096 > 300
//                              256 rows                140.9             448.4                      1 712              761.0             1 711
//                              128 rows                133.6             410.8                      1 752              796.3             1 809
//   whole prompts, slopes, whose bound is at most 3 072 tokens, or that 256-row workgroups fill not five times
//                         -> 128 rows; in a longer walk the loads that 256 rows save weigh more.  (They tie at 2 816; prompts may be shorter than
//                            their bound, and then 128 rows win: 4 of 768 under 2 048, tiles through registers, 40.6 and 37.2.)  8 prompts, the first two columns with the same inputs again and again, the others with three sets in turn:
//                              tokens                 1 024   1 536   2 560   2 816   3 072   3 328   3 584   4 096   16 x 3 072   16 x 3 584
//                              256 rows                95.6   183.5   342.2   392.1   441.2   492.0   546.9   662.2      902.6      1 085.7
//                              128 rows                88.6   165.7   340.5   394.0   449.2   509.4   562.0   689.4      917.6      1 115.4
//                              fp16, 256 rows                                         408.6           498.4   600.8
//                              fp16, 128 rows                                         405.7           509.6   623.3
//   else                  -> 256 rows.
inline PrefillShape prefill_shape_direct(int64_t units8, int heads_pow2_shift, int max_q_len, int head_dim, bool slopes, bool windowed,
                                         bool whole_prompts, int cus, int64_t key_bytes)
{
    const PrefillShape any = prefill_shape(units8, heads_pow2_shift, max_q_len, windowed, cus);
    if (windowed || any == PrefillShape::k8WavesTwoGroups) return any;
    const int64_t tiles4 = prefill_q_tiles(4, heads_pow2_shift, max_q_len), tiles8 = prefill_q_tiles(8, heads_pow2_shift, max_q_len);
    const int64_t blocks8 = units8 * tiles8;
    bool wide = head_dim == 128;
    if (whole_prompts) wide = wide && blocks8 > 5 * cus && (slopes ? max_q_len > 3072 : key_bytes >= kPrefillFarKeys);
    else if (slopes) wide = wide && 4 * blocks8 >= (tiles8 > 1 ? 7 : 8) * cus;
    else wide = wide && blocks8 >= 2 * cus && ((tiles4 > tiles8 && key_bytes >= kPrefillFarKeys) || max_q_len > 2048);
    return wide ? PrefillShape::k8Waves : PrefillShape::k4Waves;
}

// Whether tiles that go to LDS directly, from a cache, are asked for two steps ahead instead of one.  seen: tokens that a row may see, under the width of the
// block tables (and a window).  One step is a memory latency or less where few rows are computed faster than their next keys arrive, and with slopes,
// where most heads' walks end early, for the long walks that are left.  Elsewhere the buffers and instructions of the second step cost 2 to 4 %.
// Time of through registers, as it was once, over that with one step, and over that with two: geometric mean and least of random shapes (bf16 and
// fp16, 1-100 sequences, caches in turn that are no longer in the last-level cache):
//   one tile of 128 rows to a unit, at most one workgroup to a CU
//                            200-500 seen       500-1 000       1 000-2 000      2 000-4 096      beyond
//     slopes, head_dim 128  1.13 .99 | 1.12 1.02   1.09 .87 | 1.10 1.03   1.05 .81 | 1.13 1.04   1.04 .86 | 1.16 1.03    .93 .73 | 1.16 1.05
//     none, head_dim 128    1.12 .98 | 1.11 1.00   1.06 .87 | 1.09 1.03   1.01 .81 | 1.08 1.03    .92 .77 | 1.07  .99    .90 .74 | 1.09 1.00
//     none, head_dim 64     1.10 .97 | 1.07 1.00   1.04 .91 | 1.03 1.00   1.01 .85 | 1.04  .99    .97 .81 | 1.04  .97    .93 .77 | 1.03  .96
//     window, head_dim 128  1.07 .98 | 1.04  .99   1.07 .90 | 1.07 1.04   1.05 .90 | 1.11 1.08   1.06 .87 | 1.13 1.09
//   two tiles             1.10 1.04 | 1.07 1.00  1.08 1.02 | 1.06 1.00   1.08 .98 | 1.08  .98   1.08 .96 | 1.09  .98    .99 .82 | 1.12  .98
//   more workgroups, one or two tiles: 257-512 of them 1.00 .86 | 1.11 .94, beyond 1.29 .85 | 1.38 .78
//   three tiles and more, slopes, beyond 4 096: .93 .82 | 1.16 .95 (8 chunks of 512 behind 2 048 109 us and 109)
inline bool prefill_deep(int64_t units8, int heads_pow2_shift, int max_q_len, bool slopes, bool windowed, int cus, int64_t seen)
{
    const int64_t tiles4 = prefill_q_tiles(4, heads_pow2_shift, max_q_len);
    if (tiles4 > 2) return slopes && !windowed && tiles4 <= 16 && seen >= 4096;
    return units8 * tiles4 > cus || seen >= (tiles4 == 1 ? 512 : 1000);
}

}  // namespace optgqa
