// Prefill over the paged cache: several new query tokens per sequence, causal mask + ALiBi
// (Alg. 1, prompt branch: scores, bias, softmax, weighted sum), as tiled matrix-core contractions.
//
// Workgroup (4 or 8 waves, see WAVES below) = 32 (query token, head) rows per wave of one
// (sequence, KV head [x chunk of the group]) against the whole visible context, in 32-key tiles
// staged through LDS and shared by the waves.  The rows are the same tokens of every head of the group
// (head by head, or token by token: kPfByHeadTiles), so all heads of the group consume the same K/V tile (Section II: a group shares one
// key-value pair).
//
// A wave owns 32 rows.  Both contractions are computed transposed, with v_mfma_f32_32x32x16, so that
// no operand has to be transposed in registers:
//   S^T[key][row] = K Q^T      A = K rows from LDS (natural layout: lane (key L % 32, slab L / 32)
//                              needs 8 consecutive dims of its key), B = the lane's query row held in
//                              VGPRs.  The accumulator starts from the tile-invariant part of the
//                              ALiBi term, so one FMA per score finishes eq. (3).  A lane then holds,
//                              for ONE query row, 16 of the tile's 32 scores (keys 8i + 4 * slab + j in
//                              element 4i + j), which after the softmax pack straight into ...
//   O^T[dim][row] += V^T P^T   ... the B operands of the two output MFMAs of a 32-dim block, whose
//                              contraction index runs over the tile's keys in exactly that
//                              (permuted) order.  A = V^T: V lies in LDS as rows of dims (16-byte pieces
//                              of a key) and is read with the LDS transpose load (ds_read_b64_tr_b16:
//                              inside each group of 16 lanes, lane i receives element i % 4 of the
//                              8-byte chunks addressed by lanes i/4, 4 + i/4, 8 + i/4, 12 + i/4),
//                              so that a lane ends up with four consecutive keys of its dim from
//                              one instruction.
// (32x32x16 rather than 16x16x32 MFMAs: same flops per cycle, half as many matrix and LDS
// instructions per tile, and a row's scores live in 2 lanes instead of 4.  Measured on one CU, a
// SIMD overlaps such MFMAs of one wave with vector instructions of another - 16 of them and 64 FMAs take 521
// cycles together - but a wave issues at most one instruction every ~4.4 cycles and the loop is a chain of scores,
// softmax, products and a barrier, 2 090 to 2 335 cycles a tile for a pair of waves whose MFMAs take 1 536 (bf16): the instructions of a tile are
// what this kernel is tuned for.)
// Scores, sums and the output accumulate in fp32.  For the second contraction the softmax
// weights must become 2-byte values:
//   fp16: one rounding (11 significant bits); the lazily moved reference of the exponentials (see
//         decode_mma_kernels.hpp) is kept tight enough (threshold 2^14, headroom 2^2) that weights
//         stay inside fp16's range;
//   bf16: 8 significant bits are not enough for the 1e-2 output budget once the output itself is
//         rounded to bf16 (measured: 1.003e-2), so each weight is split into a bf16 head and a
//         bf16 tail and the contraction runs twice; bf16's range allows the wide lazy reference.
//
// Key order.  Without a window the tiles are walked from the diagonal BACKWARDS (newest keys
// first).  With ALiBi the bias falls as the walk goes on, so the softmax reference that the first
// tiles set stays valid (walking forwards, steep heads push it up every other tile and the
// accumulators are rescaled each time), and a tile can be judged against what has already been
// summed: when, for every row of the wave, the largest weight of the tile is below 2^-24 of the
// row's sum so far - half an ulp of that fp32 sum, a fact read off the scores, not assumed from
// the slopes - the tile's exponentials, weight packing and output MFMAs are skipped.  Each dropped
// weight is one that an fp32 "sum += w" would have rounded away by itself; a tile drops at most
// 32 of them per row (2^-19 of the row sum).  Under a positive slope the weights that could lie at the threshold
// fall from tile to tile, and the total stays within a few 2^-19 - three orders of magnitude below the compute
// budget of the stated tolerance; without one it is bounded by 2^-24 a key (2^-9 of the sum if all of 32 768
// keys lie just below the threshold).  (The definition, eq. (3)-(4), still sums every key; heads with a
// steep slope simply give most keys a weight that no fp32 sum can see.)
#pragma once
#include <type_traits>

#include "decode_mma_kernels.hpp"
#include "prefill_shape.hpp"

namespace optgqa {

// log2 of the fraction of a row's running sum below which a whole tile's weights are dropped
// (half an ulp of an fp32 sum)
#ifndef OPTGQA_PF_SKIP_LOG2
#define OPTGQA_PF_SKIP_LOG2 (-24.f)
#endif
constexpr float kPfSkipLog2 = OPTGQA_PF_SKIP_LOG2;
// tiles between a look at whether the rest of the walk still matters, at the least (2, 4 and 8 measure the same)
constexpr int kPfCheckTiles = 4;
// ... and tiles that must be left for the look to pay (rest_judged costs about 2 us; looking from 4, 12 and 16 tiles
// on: 5 chunks of up to 1 419 behind 630 110.0, 110.0 and 111.4 us, 5 prompts of 1 280 88.4, 87.9 and 89.9)
constexpr int kPfJudgeTiles = 12;
// tiles that a launch's longest possible walk must have for the kernel that looks to be taken (JUDGE).  (GPU time with it
// and without, slopes: head_dim 64, 16 / 4 heads, 3 prompts of 1 024 26.2 and 24.2 us, 3 of 1 280 31.9 and 28.7, 3 of 1 536 38.5 and
// 36.1, 12 of 1 280 64.8 and 65.3, 3 of 2 560 69.0 and 71.0; head_dim 128, 8 of 512, 32 / 8, 42.7 and 40.5, 364 to 1 093 over 8-bit
// caches, 32 / 4, 40.2 and 39.4, 5 of 1 024, 32 / 8, 64.5 and 66.0, 5 of 1 152 77.7 and 79.9, 5 of 1 280 88.6 and 94.1, 5 chunks of
// up to 1 419 behind 630 110 and 118.)
template <int D> constexpr int kPfJudgeLongest = D == 128 ? 36 : 48;
// tiles that a look which fails further on must have passed for the walk to leave them out (starting it anew costs about 3 us)
constexpr int kPfJumpTiles = 8;
// tiles that a walk must have for a wave's rows to be one head's; below, a token's heads are neighbouring rows, as they are
// in memory (slopes, always by head and never: 8 prompts of 170-512, 16 / 4 heads, head_dim 64, 14.2 and 13.8 us; 32 / 8,
// head_dim 128, 25.2 and 25.2, 8 chunks of 128 behind 300 19.3 and 19.2, of 256 behind 512 36.3 and 36.7; longer walks skip more by
// head: 4 prompts of 1 024 55.7 and 56.2, 8 chunks of 512 behind 2 048 111.5 and 116.1.  Before rows went through LDS whole, short
// walks by head lost 5 %.)
constexpr int kPfByHeadTiles = 16;
// tiles that a walk must have for two key groups to share it: below, the second group's waves end at once and the
// first walks alone.  (Sharing costs a tile beyond the diagonal, a merge through LDS and two barriers.  GPU time shared
// over alone, 32 / 8 heads, one prompt with slopes or 4 chunks of 40 behind a cache without, bf16 and fp16, 8 sets of inputs in turn:
//   tiles                       1           2           4           6           8           10          11          12          16          24
//   head_dim 128, prompt    1.26        1.15-1.17   1.09-1.12   1.04-1.07   1.00-1.03   0.97-1.03   0.98-1.02   0.95-0.99   0.92-0.95   0.90-0.93
//   head_dim 128, chunks                1.03-1.05   1.01-1.02   0.96-0.99   0.94-0.95   0.92-0.94   0.96-0.97   0.91        0.89        0.85-0.86
//   head_dim 64, prompt     1.18        1.08-1.09   1.02-1.04   0.98-0.99   0.94-0.95   0.91-0.92   0.93        0.89-0.90   0.85-0.87   0.83-0.84
//   head_dim 64, chunks                 1.02        0.96-1.00   0.93-0.95   0.91-0.92   0.88-0.89   0.92-0.94   0.86-0.88   0.83-0.84   0.80
// The lines lie where prompts tie, or a little beyond.)
template <int D> constexpr int kPfTwoGroupTiles = D == 128 ? 11 : 8;

struct PrefillParams {
    void* out;                  // [T][Hq][D] dtype
    const void* q;              // [T][Hq][D]
    const void* k_cache;        // [NB][Hkv][bs][D]
    const void* v_cache;
    const int32_t* block_tables;
    const int32_t* context_lens;
    const int32_t* cu_q_lens;   // [B + 1]
    const float* slopes;        // [Hq] or nullptr
    float scale2;               // scale * log2(e) (times k_scale for E4M3 caches)
    float out_scale;            // multiplies the output (v_scale of an E4M3 cache, else 1)
    const float* k_scales;      // E4M3 caches with one scale pair per KV head: device arrays [num_kv_heads]
    const float* v_scales;      // (then scale2 holds no k_scale and out_scale is 1), else nullptr
    int num_heads, num_kv_heads, block_size, max_blocks_per_seq;
    int num_seqs;
    int heads_per_wg;           // GH: query heads per workgroup (divides the group size, <= 16)
    int heads_pow2_shift;       // log2 of GH rounded up to a power of two (rows per workgroup >> shift: its tokens)
    int q_tiles;                // ceil(max_q_len / tokens per workgroup)
    int units;                  // num_seqs * num_kv_heads * (group / GH)
    int group;                  // query heads per KV head
    int chunks;                 // group / GH
    int units_per_seq;          // num_kv_heads * chunks
    FastDiv by_units_per_seq, by_chunks;
    FastDiv by_tiles, by_units;                     // with slopes: q_tiles and num_seqs, else ceil(units / 8) and units_per_seq
    int tiles_div, units_div;                       // those divisors
    int deep;                   // tiles are asked for two steps ahead (the host's choice of a kernel)
    int window;                 // > 0: the query at position pos sees keys pos - window < j <= pos only
    // whole-prompt variant (CONTIG): K/V come from the step's contiguous inputs, not from the cache
    const void* k_in;           // [T][Hkv][D] with token strides (elements)
    const void* v_in;
    int64_t k_in_stride, v_in_stride;
    void* k_cache_w;            // caches to store the prompt's K/V into (both or neither), else nullptr
    void* v_cache_w;
};

// Workgroup shapes (template parameters WAVES and KS; 32 rows per wave, chosen in prefill_shape.hpp):
//   8 waves            256 rows against one K/V tile, half the loads of it per row;
//   4 waves            128 rows, two workgroups to a CU: one's start and end under the other's walk;
//   8 waves, KS = 2    128 rows, the walk's tiles dealt to two groups of four waves (each its own tile
//                      buffers), whose sums are merged through LDS at the end: half as long a walk where
//                      there are too few workgroups to fill the chip (a workgroup with a short walk uses
//                      one group only, kPfTwoGroupTiles).
// With a sliding window always 4 waves: a workgroup's rows should span few keys, because every tile that
// some row's window start or causal end cuts needs the masked path (prefill_shape.hpp has both sides' times).
constexpr int kPfKeys = 32;                              // keys per tile
// LDS rows of 8-bit caches' tiles and of a wave's strip, elements: K rows padded by 8 (16-byte reads of 16 keys then
// cover all 64 banks), V rows by 16 (so do the rows a transposing load touches) - head_dim 128: 272 / 288 bytes, 64: 144 / 160
template <int D> struct PfTile {
    static constexpr int kKRow = D + 8, kVRow = D + 16;
    static constexpr int kLdsBytes = 2 * kPfKeys * (kKRow + kVRow) * 2;   // two buffers of one K and one V tile (PfDirect's are smaller)
    static constexpr int kWaveBytes = 32 * kKRow * 2;                     // a wave's 32 query (output) rows, pitched as K rows
    // a workgroup of `waves` waves in `groups` key groups
    static constexpr int lds_bytes(int waves, int groups) { return groups * kLdsBytes + waves * kWaveBytes; }
};

// Tiles of 2-byte elements are written to LDS by the memory system itself (global_load_lds_dwordx4: 64 lanes' 16-byte
// pieces to 1 KiB from the address in m0 on, lane by lane): no registers hold a tile on its way, no LDS stores, and with
// wave-uniform addresses not one vector instruction.  (Through registers - loads, 16-byte LDS stores and their addresses -
// a tile cost a wave 20 to 30 instructions.  32 / 8 heads, head_dim 128, the same caches again and again: 8 prompts of 1 024 96.8 -> 86.0 us,
// 8 chunks of 512 behind 2 048 107.5 -> 103.3, without slopes 201 -> 195, with a window of 512 65.7 -> 61.8; whole steps over caches in turn, with 128 rows
// in more launches: those chunks 113.1 -> 110.0, with the window 71.3 -> 68.7, 8 prompts of 2 560 366.7 -> 352.0.  Few rows behind long contexts lost: prefill_deep.)
// Such a load cannot pad rows, but it may bring any piece to any lane.  A tile is groups of 4 rows (head_dim 64: 8), 1 KiB and
// a pad of 16 (32) bytes each.  In a group pieces of 64 bytes - four lanes, 64 bytes of one row's, as the memory system likes
// them - lie row behind row, then the next 64 bytes of all rows:
//     offset = (column / 4) * (64 * rows) + row * 64 + (column % 4) * 16      (columns of 16 bytes; head_dim 64: column ^ 1 in rows 4-7)
// What the score MFMAs read at once (one column of 16 rows) then lies in 16 different sixteenths of the 64 banks, and so do
// the 32-byte pieces of four rows of a transposing load; and a lane's pieces are at constant distances.
template <int D> struct PfDirect {
    static constexpr int kRows = 512 / D, kGroups = 32 / kRows;           // rows of a group; groups of a tile
    static constexpr int kGroup = 1024 + (D == 128 ? 16 : 32);            // bytes from group to group
    static constexpr int kTile = kGroups * kGroup;                        // bytes of a tile (of 32 query rows, too)
    // the row of its group and the column that lane l of a load brings
    static __device__ __forceinline__ int load_row(int l) { return (l >> 2) & (kRows - 1); }
    static __device__ __forceinline__ int load_col(int l)
    {
        return D == 128 ? (l >> 4) * 4 + (l & 3) : (l >> 5) * 4 + ((l & 3) ^ ((l >> 4) & 1));
    }
    // byte offset of dims 8 * h2 .. +7 of a row, and from there to the dims 16m further on
    static __device__ __forceinline__ int row_at(int row, int h2)
    {
        return D == 128 ? (row >> 2) * kGroup + (row & 3) * 64 + h2 * 16
                        : (row >> 3) * kGroup + (row & 7) * 64 + (h2 ^ ((row >> 2) & 1)) * 16;
    }
    static constexpr int dims_at(int m) { return (m >> 1) * 64 * kRows + (m & 1) * 32; }
    // byte offset of what lane s16 of 16 addresses in a transposing load of keys 4 * h2 .. +3, dims 16 * dhalf .. +15, and
    // from there to the keys 8 * k8 and the dims 32 * db further on
    static __device__ __forceinline__ int keys_at(int s16, int dhalf, int h2)
    {
        return D == 128 ? h2 * kGroup + (s16 >> 2) * 64 + dhalf * 32 + (s16 & 3) * 8
                        : (4 * h2 + (s16 >> 2)) * 64 + dhalf * 32 + (((s16 & 3) >> 1) ^ h2) * 16 + (s16 & 1) * 8;
    }
    static constexpr int further(int k8, int db) { return k8 * (8 / kRows) * kGroup + db * 64 * kRows; }

    // DEEP: a key group's LDS holds kDeepBuffers buffers of a K and a V tile each.  The waves' query rows lie behind K and V of the first
    // tile and K of the second, where nothing is loaded before they have been read; the output rows, after the walk, from the
    // beginning on (two groups: behind what they exchange).
    static constexpr int kDeepBuffers = 4, kRowsAt = 3 * kTile;
    static constexpr int group_bytes(int group_waves)
    {
        const int tiles = 2 * kDeepBuffers * kTile, rows = kRowsAt + group_waves * PfTile<D>::kWaveBytes;
        return tiles > rows ? tiles : rows;
    }
    static constexpr int exchange_bytes(int waves, int groups) { return groups == 1 ? 0 : waves * 64 * (D / 64 * 4 * 16 + 8); }
    static constexpr int deep_lds_bytes(int waves, int groups)
    {
        const int walk = groups * group_bytes(waves / groups), out = exchange_bytes(waves, groups) + waves * PfTile<D>::kWaveBytes;
        return walk > out ? walk : out;
    }
};

// One such load, to LDS address `lds` (wave-uniform) on; from a wave-uniform base and lane offsets, or from lane addresses.
// In assembly because the compiler, which does not know which buffer a load writes, would have every later read of LDS wait
// for it; wait_direct() comes before the barrier that publishes the tile.  (m0 is an operand, which the compiler sets: it is a
// reserved register, and a statement that writes it by itself is not one that the compiler allows for.  The s_nop is the wait
// state between that and the load.)
__device__ __forceinline__ void load_direct(uint32_t lds, const unsigned char* base, uint32_t lane_off)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "{m0}"(lds), "v"(lane_off), "s"(base) : "memory");
}
__device__ __forceinline__ void load_direct(uint32_t lds, const unsigned char* lane_addr)
{
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "{m0}"(lds), "v"(lane_addr) : "memory");
}
template <int NEWER = 0> __device__ __forceinline__ void wait_direct() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NEWER) : "memory"); }

template <int DT> __device__ __forceinline__ uint32_t pack2(float lo, float hi) { return narrow2<DT>(lo, hi); }

typedef float f32x16 __attribute__((ext_vector_type(16)));
// v_mfma_f32_32x32x16: A lane (row L % 32, k-slab L / 32) holds k = 8 * slab .. + 7, B likewise
// for its column; C / D lane (column L % 32, half L / 32) holds rows 8i + 4 * half + j in
// element 4i + j (i, j = 0..3).
template <int DT> __device__ __forceinline__ f32x16 mfma32(uint4 a, uint4 b, f32x16 c);
template <> __device__ __forceinline__ f32x16 mfma32<kF16>(uint4 a, uint4 b, f32x16 c)
{
    typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x16 mfma32<kBF16>(uint4 a, uint4 b, f32x16 c)
{
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// what this wave wrote to LDS is there for its other lanes (LDS instructions of a wave complete in order; the compiler
// keeps theirs across this)
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int DT> struct PfSoftmax;
template <> struct PfSoftmax<kF16> {
    static constexpr float kThreshold = 14.f, kHeadroom = 2.f;
    static constexpr bool kSplitWeights = false;
};
template <> struct PfSoftmax<kBF16> {
    static constexpr float kThreshold = kRescaleThreshold, kHeadroom = kRescaleHeadroom;
    static constexpr bool kSplitWeights = true;
};

#ifndef OPTGQA_PF_WAVES_PER_SIMD
#define OPTGQA_PF_WAVES_PER_SIMD 2
#endif
// KV8: the caches hold 1-byte E4M3 codes with per-tensor scales (k_scale folded into scale2,
// v_scale into out_scale on the host); the loader threads widen them to DT - exactly - on the
// way into LDS, everything after that is unchanged.
//
// CONTIG: the whole prompt is new and nothing of it is in the cache yet (Alg. 1, prompt branch with
// empty caches): the context of sequence b is its own cu_q_lens[b+1] - cu_q_lens[b] tokens, and
// K / V tiles are fetched from the contiguous inputs k_in / v_in (token strides) instead of
// through the block table.  With k_cache_w / v_cache_w set, the workgroups of a KV head's first
// head chunk also store their own tokens' K / V rows into the paged caches (Alg. 1, the
// cache-store step), so the step needs no separate cache-write launch.
//
// STEP: one prefill step over a cache that already holds the earlier tokens (Alg. 1: the cache-store
// step, then the attention): the n_b new tokens of sequence b have their K / V rows in k_in / v_in
// (token cu_q_lens[b] + i = position context_lens[b] - n_b + i) and NOT yet in the cache.  A key
// below the first new position is fetched through the block table, a key at or above it from the
// inputs - chosen per key, both addresses are always valid - and, as with CONTIG, the workgroups of
// a KV head's first head chunk store their own tokens' rows into the caches.  No workgroup reads
// a cache row that this launch writes.
//
// JUDGE: slopes are given and walks may be long enough to be ended early (rest_judged).  A switch because the code of it,
// even where it never runs, costs the loop around it its instruction order (no slopes, 5 prompts of 512, 16 / 4 heads,
// head_dim 64, bf16: 15.3 us without it in the kernel, 16.4 with; 3 of 1 024: 24.3 and 27.1; 8 chunks of 512 behind 2 048,
// 32 / 8 heads, head_dim 128: 217.8 and 220.2), and because a look costs what walks of up to kPfJudgeLongest tiles cannot
// earn back (slopes, prompts of 512: 3 with 16 / 4 heads, head_dim 64, 12.1 and 13.6; 8 with 32 / 8, head_dim 128, 40.5 and 42.7).
//
// DEEP: tiles are asked for two steps ahead instead of one (prefill_shape.hpp says where).
template <int DT, bool KV8, bool WIN, bool CONTIG, bool JUDGE, int D, int WAVES, int KS, bool DEEP, bool STEP>
__device__ __forceinline__ void prefill_body(const PrefillParams& p)
{
    static_assert(!(JUDGE && WIN), "a windowed walk is short: never judged");
    static_assert((WAVES == 4 && KS == 1) || (WAVES == 8 && !WIN && (KS == 1 || KS == 2)), "4 waves; without a window also 8, or 8 in two key groups");
    constexpr int kPfWaves = WAVES / KS, kPfRows = kPfWaves * 32;   // of one key group: its waves, and the workgroup's rows
    static_assert(!(CONTIG && (KV8 || WIN)), "the whole-prompt variant reads 2-byte inputs, full causal mask");
    static_assert(!(DEEP && (KV8 || CONTIG)), "tiles that go to LDS directly, from a cache");
    static_assert(!(STEP && (KV8 || WIN || CONTIG)), "the one-call step runs over 2-byte caches, full causal mask");
    static_assert(D == 128 || D == 64, "head_dim 64 or 128");
    constexpr int kPfKRow = PfTile<D>::kKRow, kPfVRow = PfTile<D>::kVRow;
    constexpr int kQ = D / 16;                          // score MFMAs per tile (16 dims each)
    constexpr int kDB = D / 32;                         // 32-dim blocks of the output
    constexpr int kCPR = D / 8;                         // 16-byte (8-element) column pieces per row
    constexpr int kKPT = kPfKeys * (D / 8) / (kPfWaves * 32);   // consecutive keys a loader thread moves per tile (half the threads per tensor)
    constexpr int ES = KV8 ? 1 : 2;                     // bytes per cache element
    constexpr bool DIRECT = !KV8;                       // tiles go to LDS as they are (8-bit codes pass through registers, which widen them)
    typedef PfDirect<D> Direct;
    // tile buffers, each a K tile followed by a V tile: PfDirect's, or two of [32][kPfKRow] and [32][kPfVRow]
    constexpr int kKTile = DIRECT ? Direct::kTile / 2 : kPfKeys * kPfKRow;
    constexpr int kBuf = kKTile + (DIRECT ? Direct::kTile / 2 : kPfKeys * kPfVRow);
    constexpr int kBuffers = DEEP ? Direct::kDeepBuffers : 2, kLead = DEEP ? 2 : 1;      // kLead: steps that a tile is asked for ahead
    static_assert(kLead < kBuffers && (kBuffers & (kBuffers - 1)) == 0, "K tiles j + 1 .. j + 1 + kLead, V tiles j .. j + kLead; a power of two");
    constexpr int kGroupLds = DEEP ? Direct::group_bytes(kPfWaves) / 2 : kBuffers * kBuf;        // a key group's
    static_assert(DEEP || 2 * 2 * kBuf <= PfTile<D>::kLdsBytes, "both layouts fit");
    static_assert(Direct::kTile <= PfTile<D>::kWaveBytes, "a wave's query rows fit its strip");
    extern __shared__ __attribute__((aligned(16))) uint16_t tile_lds[];          // prefill_lds_bytes<D>(WAVES, KS, DEEP)
    __shared__ float vote[3][WAVES];                          // rest_judged
    __shared__ int nearest_bad;
    __shared__ uint32_t least_norm2;

    // ---- which rows -----------------------------------------------------------------------
    // XCD-aware order: workgroups go to XCD (flat id % 8); all query tiles of one (sequence, KV
    // head) unit are given the same residue so that its K/V stay in one XCD's L2 (but for the order by
    // length below, where that holds with a multiple of 8 KV heads x head chunks only: with 2, 3 or 4 a unit's tiles lie
    // on 4, 8 or 2 XCDs, and its keys are read from memory more than once, which a kernel bound by its matrix
    // instructions does not show - 24 ragged chunks without slopes, 8 / 2 heads: 235 -> 155 us, 24 / 3: 542 -> 449,
    // 16 / 4: 416 -> 295, 32 / 8: 681 -> 586 with the order by length).
    // Longest first: the hardware hands workgroups to free slots in id order, so the workgroups that
    // will run longest should have the lowest ids and the short ones fill the tail of the launch.
    // A later query tile sees more keys; and, walking backwards from the diagonal, a head with a
    // steep ALiBi slope skips most of its tiles while one with a shallow slope skips none - slopes
    // fall with the head number in every usual recipe, so the units are taken from the last KV head
    // down (a wrong guess costs nothing but the order).  Consecutive units, which then share a KV
    // head, are dealt to different XCDs (rotation by the row of eight).
    const int xcd = blockIdx.x & 7, w = blockIdx.x >> 3;
    const int Hq = p.num_heads, Hkv = p.num_kv_heads, bs = p.block_size;
    const int bs_shift = __builtin_ctz(bs);
    const int GH = p.heads_per_wg, gshift = p.heads_pow2_shift;
    const int G = p.group, chunks = p.chunks, units_per_seq = p.units_per_seq;
    const int tshift = __builtin_ctz(kPfRows) - gshift, tokens_per_wg = 1 << tshift;
    // Without slopes nothing is skipped and the query tile's position alone decides the length: with up to
    // 64 sequences (a lane each) workgroup number n takes the (n / units per sequence)-th of all (sequence,
    // query tile) pairs in falling order of their last position, counted in query tiles.  (Ragged chunks, 6
    // sequences of 333-777 new tokens behind 5-2999 cached: by query tile alone the launch's longest
    // workgroup started in its middle.)
    const bool by_head = p.slopes != nullptr;
    int b, gu, qt, cu0, n_b, ctx_len;
    if (KS == 1 && !WIN && !by_head && p.num_seqs <= 64) {       // (two key groups: all workgroups start at once anyway)
        const int rank = p.by_units_per_seq.div(blockIdx.x);
        const int l = threadIdx.x & 63, lc = min(l, p.num_seqs - 1);
        const int c0 = p.cu_q_lens[lc], n = p.cu_q_lens[lc + 1] - c0, len = CONTIG ? n : p.context_lens[lc];
        const int tiles = l < p.num_seqs && n > 0 ? (n + tokens_per_wg - 1) >> tshift : 0;
        const int before = max(len - n, 0) >> tshift;      // query tiles' worth of cached tokens
        // the pairs that end at or beyond position x (in query tiles): tile q of a sequence ends at before + q + 1
        auto count = [&](int x) __attribute__((always_inline)) {
            return wave_sum(min(tiles, max(before + tiles - x + 1, 0)));
        };
        if (count(1) <= rank) return;
        int lo = 1, hi = wave_max(tiles > 0 ? before + tiles : 0) + 1;   // count(lo) > rank >= count(hi) = 0
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (count(mid) > rank) lo = mid;
            else hi = mid;
        }
        // the rank's pair ends at lo: of those that do, in order of the sequences
        uint64_t at = __builtin_amdgcn_ballot_w64(before < lo && lo <= before + tiles);
        for (int skip = rank - count(lo + 1); skip > 0; --skip) at &= at - 1;
        b = __builtin_ctzll(at);
        qt = lo - 1 - __builtin_amdgcn_readlane(before, b);
        cu0 = __builtin_amdgcn_readlane(c0, b);
        n_b = __builtin_amdgcn_readlane(n, b);
        ctx_len = __builtin_amdgcn_readlane(len, b);
        gu = blockIdx.x - rank * units_per_seq;
    } else {
        // w: row of eight units, query tile; the unit: sequence, KV head x chunk (by head: the units of a KV head in a row)
        const int quot = p.by_tiles.div(w), rest = w - quot * p.tiles_div;
        const int urow = by_head ? quot : rest;
        qt = p.q_tiles - 1 - (by_head ? rest : quot);
        const int ui = urow * 8 + ((xcd - urow) & 7);
        if (ui >= p.units) return;
        const int uq = p.by_units.div(ui), ur = ui - uq * p.units_div;
        b = by_head ? ur : uq;
        gu = by_head ? units_per_seq - 1 - uq : ur;
        cu0 = p.cu_q_lens[b];
        n_b = p.cu_q_lens[b + 1] - cu0;
        ctx_len = CONTIG ? n_b : p.context_lens[b];
    }
    const int g = p.by_chunks.div(gu);
    const int h0 = g * G + (gu - g * chunks) * GH;
    const int tq0 = qt * tokens_per_wg;
    if (tq0 >= n_b) return;
    const int L = ctx_len;
    const int pos0 = L - n_b;                                   // position of the sequence's first new token
    const int kmax = pos0 + min(tq0 + tokens_per_wg, n_b);      // keys 0 .. kmax-1 are visible to some row
    const int ntiles = (kmax + kPfKeys - 1) / kPfKeys;
    // Sliding window (Alg. 1, local mask): the workgroup's first row sits at pos0 + tq0 and sees no
    // key before kmin, later rows see even fewer of the early keys, so the tiles before kmin's are
    // never read.
    // (WIN is a compile-time switch so that the plain causal kernel carries none of this)
    const int W = WIN ? p.window : 0;
    const int kmin = W > 0 ? max(pos0 + tq0 - W + 1, 0) : 0;
    const int kt0 = kmin / kPfKeys;

    // wg_wave: the wave's number in the workgroup; kw: its key group; wave, tid: its and its thread's number in that
    const int lane = threadIdx.x & 63;
    const int wg_wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kw = KS == 1 ? 0 : wg_wave / kPfWaves, wave = KS == 1 ? wg_wave : wg_wave % kPfWaves;
    const int tid = KS == 1 ? threadIdx.x : threadIdx.x % (kPfWaves * 64);
    const int n32 = lane & 31, h2 = lane >> 5;
    // two key groups: whether they share the walk (log2 of the groups that do), and the waves that stay
    const int share = KS == 1 ? 0 : ntiles >= kPfTwoGroupTiles<D> ? 1 : 0;        // workgroup-uniform
    const int nwaves = kPfWaves << share;
    if (KS == 2 && wg_wave >= nwaves) return;

    // paged: the KV head's offset inside a block; CONTIG: the sequence's token 0, KV head g
    const unsigned char* __restrict__ kc = CONTIG
        ? static_cast<const unsigned char*>(p.k_in) + (cu0 * p.k_in_stride + (int64_t)g * D) * 2
        : static_cast<const unsigned char*>(p.k_cache) + (int64_t)g * bs * D * ES;
    const unsigned char* __restrict__ vc = CONTIG
        ? static_cast<const unsigned char*>(p.v_in) + (cu0 * p.v_in_stride + (int64_t)g * D) * 2
        : static_cast<const unsigned char*>(p.v_cache) + (int64_t)g * bs * D * ES;
    const int32_t* __restrict__ table = p.block_tables + (int64_t)b * p.max_blocks_per_seq;
    const int64_t block_stride = (int64_t)Hkv * bs * D;

    // STEP: the sequence's first new token, KV head g, in the inputs
    const unsigned char* __restrict__ kin = !STEP ? kc
        : static_cast<const unsigned char*>(p.k_in) + (cu0 * p.k_in_stride + (int64_t)g * D) * 2;
    const unsigned char* __restrict__ vin = !STEP ? vc
        : static_cast<const unsigned char*>(p.v_in) + (cu0 * p.v_in_stride + (int64_t)g * D) * 2;

    // CONTIG / STEP: this workgroup's own tokens' K / V rows of head g go into the caches, as 16-byte
    // pieces (kCPR per row and tensor; 2 * kCPR threads to a token, K row then V row).  The first kOwnBatch
    // tokens of every thread are loaded here, in front of the first tile fetch, and
    // stored once that tile has landed - one memory latency shared with the fetch instead of a
    // load-then-store loop of its own in front of or behind the walk (a workgroup of 256 rows has the CU to
    // itself, so such a loop is not overlapped by anything: measured 2 us per workgroup round);
    // whatever is left (more than kOwnBatch * own_step tokens per workgroup) goes out behind the output.
    constexpr int kOwnBatch = 4;
    typedef uint32_t own_u32x4 __attribute__((ext_vector_type(4)));
    const int own_tokens = ((CONTIG || STEP) && p.k_cache_w && gu == g * chunks) ? min(tokens_per_wg, n_b - tq0) : 0;
    const int own_step = nwaves * 64 / (2 * kCPR);
    // token t of the workgroup's, the piece of thread `thread`
    auto own_src = [&](int thread, int t) __attribute__((always_inline)) {
        const bool is_v = (thread / kCPR) & 1;
        const uint32_t row = (uint32_t)((is_v ? p.v_in_stride : p.k_in_stride) * 2);
        return reinterpret_cast<const own_u32x4*>((is_v ? vin : kin) + 16 * (thread % kCPR) + (uint64_t)(uint32_t)(tq0 + t) * row);
    };
    auto own_blk_of = [&](int t) __attribute__((always_inline)) {
        return table[(pos0 + tq0 + t) >> bs_shift];              // position in the sequence (CONTIG: pos0 == 0)
    };
    typedef __attribute__((address_space(1))) unsigned char* global_byte_ptr;   // (device memory, which the asm would hide)
    // this thread's piece of row 0 of block 0, KV head g
    auto own_cache = [&](int thread) __attribute__((always_inline)) {
        uint64_t k = reinterpret_cast<uint64_t>(p.k_cache_w), v = reinterpret_cast<uint64_t>(p.v_cache_w);
        asm volatile("" : "+s"(k), "+s"(v));                     // (both by scalar loads: a choice of arguments is fetched like data, behind the tiles)
        const bool is_v = (thread / kCPR) & 1;
        return (global_byte_ptr)(is_v ? v : k) + (int64_t)g * bs * D * 2 + 16 * (thread % kCPR);
    };
    auto own_dst = [&](global_byte_ptr cache, int t, int blk) __attribute__((always_inline)) {
        const int tok = pos0 + tq0 + t;
        return (__attribute__((address_space(1))) own_u32x4*)(cache + (uint64_t)(uint32_t)blk * (uint32_t)(block_stride * 2)
                                            + (uint32_t)((tok & (bs - 1)) * (D * 2)));
    };
    // ---- tiles: the first half of the waves fetches K, the second V -----------------------------------------
    const bool k_loader = wave < kPfWaves / 2;                   // wave-uniform
    const int l_ahead = k_loader ? 1 : 0;                        // K tiles run one tile ahead of V tiles (below)
    const unsigned char* __restrict__ l_src = k_loader ? kc : vc;
    const int64_t l_row = CONTIG ? (k_loader ? p.k_in_stride : p.v_in_stride) * 2 : D * ES;   // bytes from key to key
    // STEP: the first new token's row, and the inputs' bytes from token to token
    const unsigned char* const l_in = k_loader ? kin : vin;
    const uint32_t l_in_row = STEP ? (uint32_t)((k_loader ? p.k_in_stride : p.v_in_stride) * 2) : 0u;
    const uint32_t l_blk_bytes = (uint32_t)(block_stride * ES);                   // < 2^32: one block of all KV heads
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // native vectors: plain loads and stores
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    // Key groups: of every two consecutive tiles of the walk each group takes one.  The walk is made a
    // multiple of two long by starting it beyond the diagonal, where the causal mask hides every key.
    const int pad = KS == 1 ? 0 : (ntiles - kt0) & share;
    const int last_tile = ntiles - 1 + pad;                       // >= kt0
    const int nt = ntiles - kt0 + pad;                            // tiles this workgroup walks
    const int steps = nt >> share;                                // ... in steps of a tile for each group
    // the tile of the walk's i-th step (i past the end: the last one again)
    auto tile_of = [&](int i) __attribute__((always_inline)) {
        const int ic = min((i << share) + kw, nt - (1 << share) + kw);
        return last_tile - ic;                                    // from the diagonal backwards
    };
    // A tile's place in LDS: the j-th tile of the walk sits in buffer j % kBuffers.
    const int group_base = kw * kGroupLds;
    auto tile_base = [&](int j) __attribute__((always_inline)) { return group_base + (j & (kBuffers - 1)) * kBuf; };
    auto tile_base_v = [&](int j) __attribute__((always_inline)) { return group_base + (j & (kBuffers - 1)) * kBuf + kKTile; };

    // Everything a workgroup starts with is asked for before anything is waited for: the block numbers of
    // the first tiles, the query rows, this workgroup's own new rows, then the first two tiles.  (What the source
    // says here the compiler does not keep by itself: a value that it widens, scales or selects where it is loaded is
    // waited for there, and a load may sink to its use.  The few lines of asm below hold such places: one memory round trip
    // before the first tile instead of three, five where new rows are stored - 8 prompts of 2 560 383.9 -> 371.6 us, with the
    // divisions by FastDiv.)

    // ---- DIRECT: 1 KiB groups of a tile by loads to LDS; a loader wave's groups are consecutive keys of one block ----------
    constexpr int kWaveGroups = Direct::kGroups / (kPfWaves / 2);
    static_assert(kWaveGroups * Direct::kRows <= 16, "a wave's keys of a tile lie in one block");
    const int d_first = kWaveGroups * Direct::kRows * (k_loader ? wave : wave - kPfWaves / 2);     // the first of them
    const uint32_t d_off = (uint32_t)Direct::load_row(lane) * (uint32_t)l_row + 16u * (uint32_t)Direct::load_col(lane);
    const bool far_rows = CONTIG && l_row >= (1ll << 29);        // (32-bit lane offsets reach seven rows)
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)tile_lds;
    const uint32_t d_lds = lds0 + 2 * (k_loader ? 0 : kKTile) + (uint32_t)(d_first / Direct::kRows * Direct::kGroup);
    // A lane holds one of the 64 block numbers from d_block down, so that a tile costs a lane read instead of a load.
    int d_block = 0, d_table = 0;
    auto read_table = [&](int block) __attribute__((always_inline)) {
        d_block = block;
        d_table = table[max(block - lane, 0)];
    };
    if constexpr (DIRECT && !CONTIG) read_table(min(tile_of(0) * kPfKeys + d_first, kmax - 1) >> bs_shift);
    // The tile of the walk's i-th step into that step's buffer (this wave's groups of K, or of V).  Every key of it is read, visible
    // or not; rows past the sequence's last key, which only the first tile has, re-read that one.  `head`: one of the first two tiles.
    auto direct_tile = [&](int i, auto head) __attribute__((always_inline)) {
        constexpr bool HEAD = decltype(head)::value;             // (later tiles: i < steps, and all of their keys exist)
        const int key0 = (HEAD ? tile_of(i) : last_tile - (i << share) - kw) * kPfKeys, key = key0 + d_first;
        const uint32_t lds = d_lds + 2 * tile_base(i);
        const unsigned char* base = l_src;
        if (CONTIG) {
            base += (uint64_t)(uint32_t)key * (uint32_t)l_row;
        } else {
            const int block = (HEAD ? min(key, kmax - 1) : key) >> bs_shift;
            if (__builtin_expect(!held_blocks_reach(d_block, block), 0)) {
                read_table(block);
                asm volatile("" : "+v"(d_table));                // (waited for here, not on the way that reads no table)
            }
            base += (uint64_t)(uint32_t)__builtin_amdgcn_readlane(d_table, d_block - block) * l_blk_bytes + (uint32_t)((key & (bs - 1)) * (D * ES));
        }
        if (HEAD || __builtin_expect((CONTIG && far_rows) || (STEP && key0 + kPfKeys > pos0), 0)) {     // workgroup-uniform
            // lane addresses.  STEP: a key at or above the first new position comes from the inputs, one below through the table
#pragma unroll
            for (int n = 0; n < kWaveGroups; ++n) {
                const int k = min(key + n * Direct::kRows + Direct::load_row(lane), kmax - 1);
                const unsigned char* a = CONTIG ? l_src + (uint64_t)(uint32_t)k * (uint32_t)l_row
                                                : base + (int64_t)((k & (bs - 1)) - (key & (bs - 1))) * (D * ES);
                if (STEP && k >= pos0) a = l_in + (uint64_t)(uint32_t)(k - pos0) * l_in_row;
                load_direct(lds + n * Direct::kGroup, a + 16 * Direct::load_col(lane));
            }
        } else {
#pragma unroll
            for (int n = 0; n < kWaveGroups; ++n)
                load_direct(lds + n * Direct::kGroup, base + (uint64_t)(n * Direct::kRows) * (uint32_t)l_row, d_off);
        }
    };

    // ---- 8-bit caches: through registers, which widen the codes.  A thread moves the same 8-code column piece of kKPT
    // consecutive keys (kCPR lanes cover one row).  One register stage: while tile t is computed, the loader's next tile sits in the other LDS
    // buffer and the one after it is on its way to registers; the block id of the next tile to
    // fetch is read one fetch earlier, so a fetch never waits for the table.  Fetches past the last
    // tile re-read it (cache hits): no branches around loads, which keeps the compiler's load
    // counting exact.
    const int ld = k_loader ? tid : tid - kPfWaves * 32;
    const int l_group = ld / kCPR, l_chunk = ld % kCPR;          // keys kKPT*group .. , dims 8*chunk ..
    const int l_pitch = k_loader ? kPfKRow : kPfVRow;
    const int l_dst = kKPT * l_group * l_pitch + 8 * l_chunk;
    u32x2 stage[kKPT];                                           // 8 codes of a key each
    auto load_blk = [&](int i) __attribute__((always_inline)) {
        // the keys of a group share a block (groups are aligned, clamping keeps the block)
        const int key = min(tile_of(i) * kPfKeys + kKPT * l_group, kmax - 1);
        return table[key >> bs_shift];
    };
    int blk_first = 0, blk_second = 0, blk_next = 0;
    if constexpr (!DIRECT) {
        blk_first = load_blk(0), blk_second = load_blk(1);
        blk_next = load_blk(2);
    }
    // (address arithmetic kept short on purpose - this loop pays for every instruction: one 64-bit
    // multiply-add for the block, one shift-add for the first row, then per key a clamp and a shift-add;
    // rows past the sequence's last key re-read that key, which lies in the same block)
    const unsigned char* const l_lane = l_src + 8 * l_chunk * ES;                 // this lane's column piece
    auto fetch_from = [&](u32x2 (&stage)[kKPT], int i, int blk) __attribute__((always_inline)) {
        const int key0 = min(tile_of(i) * kPfKeys + kKPT * l_group, kmax - 1);
        const int rmax = kmax - 1 - key0;                         // >= 0; < kKPT - 1 only at the sequence's end
        const unsigned char* base = l_lane + (uint64_t)(uint32_t)blk * l_blk_bytes + (uint32_t)((key0 & (bs - 1)) * (D * ES));
#pragma unroll
        for (int j = 0; j < kKPT; ++j) stage[j] = *reinterpret_cast<const u32x2*>(base + (uint32_t)(min(j, rmax) * (D * ES)));
    };
    auto fetch_tile = [&](u32x2 (&stage)[kKPT], int i) __attribute__((always_inline)) {
        fetch_from(stage, i, blk_next);
        blk_next = load_blk(i + 1);
    };
    auto store_tile = [&](const u32x2 (&stage)[kKPT], int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kKPT; ++j) {
            const uint4 x = widen8_e4m3<DT>(stage[j][0], stage[j][1]);
            *reinterpret_cast<u32x4*>(&tile_lds[(k_loader ? tile_base(buf) : tile_base_v(buf)) + l_dst + j * l_pitch]) = u32x4{x.x, x.y, x.z, x.w};
        }
    };

    own_u32x4 own[kOwnBatch];
    int own_blk[kOwnBatch];
    if (own_tokens > 0) {                                        // workgroup-uniform
#pragma unroll
        for (int c = 0; c < kOwnBatch; ++c) {
            const int t = min((int)threadIdx.x / (2 * kCPR) + c * own_step, own_tokens - 1);
            own[c] = *own_src(threadIdx.x, t);
            own_blk[c] = own_blk_of(t);
        }
    }

    // This lane's query row (row n32 of the wave's 32): B operand of the score MFMAs (dims
    // 16m + 8h2 .. +7, m = 0..7), its position, slope and validity.
    // Waves w and w + 4 of a workgroup share a SIMD, so with 8 waves the upper four take the row blocks in
    // reverse order (the first head's rows, with the steepest slope, beside the last head's).
    const int row_block = wg_wave < 4 ? wg_wave : KS == 1 ? 11 - wg_wave : 7 - wg_wave;
    uint4 qb[kQ];
    float posf, lof, slope2, m_ref, lsum;
    bool row_ok, started;
    // (with slopes, where the walk is worth it, a wave's rows are consecutive tokens of one head, so that it skips by
    // that head's slope and not by the shallowest of the group's)
    const bool rows_by_head = by_head && ntiles - kt0 >= kPfByHeadTiles;
    const int row_tshift = rows_by_head ? 0 : gshift, row_tmask = rows_by_head ? tokens_per_wg - 1 : -1;
    const int row_hshift = rows_by_head ? tshift : 0, row_hmask = rows_by_head ? -1 : (1 << gshift) - 1;
    struct Row { int token, head; bool ok; };                    // new token (clamped), head of the chunk (clamped), whether it exists
    auto row_at = [&](int r) __attribute__((always_inline)) {    // row r of the wave's 32
        const int row = 32 * row_block + r;
        const int ti = tq0 + ((row >> row_tshift) & row_tmask);
        const int head = (row >> row_hshift) & row_hmask;
        return Row{min(ti, n_b - 1), min(head, GH - 1), ti < n_b && head < GH};
    };
    const int64_t rows_base = ((int64_t)cu0 * Hq + h0) * (D * 2);              // bytes, of q and of out: the sequence's first new token
    auto row_offset = [&](const Row& row) __attribute__((always_inline)) {   // bytes, from there
        return (uint64_t)(uint32_t)row.token * (uint32_t)(Hq * (D * 2)) + (uint32_t)(row.head * (D * 2));
    };
    // The query rows come, and the output rows leave, whole rows at a time through an LDS strip of the wave's own (DIRECT: the
    // query rows like a tile, without passing through registers).  (From and to the operand layout directly, 64 lanes touch 32 rows of 16 or 32 bytes each:
    // a line per lane, and the memory pipeline's time for such lines is what a workgroup pays before and behind its walk.
    // 32 / 8 heads, head_dim 128: 8 chunks of 512 behind 2 048 121.1 -> 114.0 us, 8 prompts of 2 560 398.8 -> 383.9, 8 chunks
    // of 512 with a window of 512 74.6 -> 71.2; 5 prompts of 3-301, 16 / 4 heads, head_dim 64: 9.6 -> 9.3.)
    const int q_strip = DEEP ? 2 * group_base + Direct::kRowsAt + wave * PfTile<D>::kWaveBytes
                             : KS * PfTile<D>::kLdsBytes + wg_wave * PfTile<D>::kWaveBytes;               // bytes
    uint16_t* const strip = tile_lds + (DEEP ? Direct::exchange_bytes(WAVES, KS) + wg_wave * PfTile<D>::kWaveBytes : q_strip) / 2;     // of the output rows
    const unsigned char* const qp = static_cast<const unsigned char*>(p.q) + rows_base;
    u32x4 q_stage[kQ];                                           // (not DIRECT)
    {
        const Row mine = row_at(n32);
        row_ok = mine.ok;
        const int pos = pos0 + mine.token, hc = mine.head;
        posf = (float)pos;
        lof = W > 0 ? (float)(pos - W) : -1.f;                   // keys above this one are inside the window
        slope2 = by_head ? p.slopes[h0 + hc] : 0.f;              // (scaled below: here that would wait for it)
        m_ref = 0.f;                                             // set by the first tile in which the row sees a key
        // a row that does not exist never wants a tile: its sum is already beyond anything
        started = !row_ok;
        lsum = row_ok ? 0.f : INFINITY;
        if constexpr (!DIRECT) {
#pragma unroll
            for (int m = 0; m < kQ; ++m)
                q_stage[m] = *reinterpret_cast<const u32x4*>(qp + row_offset(row_at((64 / kCPR) * m + lane / kCPR)) + 16 * (lane % kCPR));
        }
    }
    asm volatile("" ::: "memory");                               // (asked for here, before the tiles' block numbers are waited for)
    u32x2 stage_first[kKPT];
    if constexpr (DIRECT) {
        const uint32_t lds = lds0 + q_strip;
#pragma unroll
        for (int n = 0; n < Direct::kGroups; ++n)
            load_direct(lds + n * Direct::kGroup, qp + row_offset(row_at(n * Direct::kRows + Direct::load_row(lane))) + 16 * Direct::load_col(lane));
        direct_tile(0, std::true_type{});
        if (k_loader) direct_tile(1, std::true_type{});          // wave-uniform
        wait_direct();
        const unsigned char* const mine = reinterpret_cast<const unsigned char*>(tile_lds) + q_strip + Direct::row_at(n32, h2);
#pragma unroll
        for (int m = 0; m < kQ; ++m) qb[m] = *reinterpret_cast<const uint4*>(mine + Direct::dims_at(m));
    } else {
        fetch_from(stage_first, 0, blk_first);
        fetch_from(stage, 1, blk_second);
#pragma unroll
        for (int m = 0; m < kQ; ++m)
            *reinterpret_cast<u32x4*>(strip + ((64 / kCPR) * m + lane / kCPR) * kPfKRow + 8 * (lane % kCPR)) = q_stage[m];
        wave_lds_fence();
#pragma unroll
        for (int m = 0; m < kQ; ++m) qb[m] = *reinterpret_cast<const uint4*>(strip + n32 * kPfKRow + 16 * m + 8 * h2);
    }
    {
        const uint32_t keep = row_ok ? 0xffffffffu : 0u;
#pragma unroll
        for (int m = 0; m < kQ; ++m) qb[m] = make_uint4(qb[m].x & keep, qb[m].y & keep, qb[m].z & keep, qb[m].w & keep);
    }
    asm volatile("" : "+v"(slope2));
    slope2 = row_ok ? slope2 * kLog2e : 0.f;
    // score scale (base 2) and output scale of this workgroup's KV head
    const float scale2 = KV8 && p.k_scales ? p.scale2 * p.k_scales[g] : p.scale2;
    const float out_scale = KV8 && p.v_scales ? p.v_scales[g] : p.out_scale;
    // slope * (offset of the lane's e-th key from its first key in a tile) / score scale: the part of
    // the ALiBi term that does not change from tile to tile, as the score MFMAs' starting value
    f32x16 key_bias;
    {
        const float per_key = slope2 / scale2;
#pragma unroll
        for (int e = 0; e < 16; ++e) key_bias[e] = per_key * (float)(8 * (e >> 2) + (e & 3));
    }
    f32x16 acc[kDB];                                             // O^T: dims 32db + 8i + 4h2 + j of row n32 in element 4i + j
#pragma unroll
    for (int db = 0; db < kDB; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[db][e] = 0.f;

    // ---- S^T = K Q^T : element 4i + j = score of key 32kt + 8i + 4h2 + j against row n32
    // (the accumulator starts from the tile-invariant part of the ALiBi term, already divided by the
    // score scale, so that one FMA per score finishes eq. (3))
    const int k_at = DIRECT ? Direct::row_at(n32, h2) / 2 : n32 * kPfKRow + 8 * h2;
    // `between`: what is issued behind the reads of the first four operands.  (A step's loads to LDS: in front of all reads
    // they delay the MFMAs, behind the MFMAs the softmax.  Two key groups, whose waves issue four a step, one chunk of 512 behind 8 192,
    // slopes: 134 us in front, 119 behind two reads, 116 behind four; behind the MFMAs everything is 2-5 % slower.)
    auto scores = [&](int buf, auto between) __attribute__((always_inline)) {
        f32x16 st = key_bias;
        auto read = [&](int m) __attribute__((always_inline)) {
            return *reinterpret_cast<const uint4*>(&tile_lds[tile_base(buf) + k_at + (DIRECT ? Direct::dims_at(m) / 2 : 16 * m)]);
        };
        uint4 ka[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) ka[m] = read(m);
        between();
#pragma unroll
        for (int m = 0; m < kQ; ++m) st = mfma32<DT>(m < 4 ? ka[m & 3] : read(m), qb[m], st);
        return st;
    };
    // kt: the tile's number along the context; buf: its number in the walk (LDS buffer buf % kBuffers)
    auto softmax_pv = [&](int kt, int buf, f32x16 st, auto masked) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked)::value;
        // ---- bias, causal mask, lazily referenced exponentials (eq. (3), (4)) --------------------
        // x = score - reference, formed directly: st*scale2 + slope2*key + (-slope2*pos - m_ref)
        const float k0 = (float)(kt * kPfKeys + 4 * h2);
        const float cm = -fmaf(slope2, posf, m_ref);
        const float b0 = fmaf(slope2, k0, cm);                   // bias - reference of this lane's first key
        float x[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            x[e] = fmaf(st[e], scale2, b0);
            if (MASKED) {
                const float keyf = k0 + (float)(8 * (e >> 2) + (e & 3));
                const bool visible = WIN ? (keyf <= posf && keyf > lof) : keyf <= posf;
                x[e] = visible ? x[e] : -INFINITY;
            }
        }
        float mx = x[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, x[e]);
        {
            // Walking backwards, the weights of a tile can be judged against what is already summed:
            // below 2^kPfSkipLog2 of the row's sum (this lane's half of it, which is no more) for
            // every row of the wave, the tile changes no bit that the accumulators keep.
            const float room = __builtin_amdgcn_logf(lsum) + kPfSkipLog2;        // log2; -inf before the row's first key
            if (__builtin_amdgcn_ballot_w64(mx > room) == 0) return;
        }
        // Has the row seen a key yet?  Walking backwards from the diagonal, a row's first visible key
        // may lie in a later tile of the walk than another row's.
        const bool first = !started;
        if (__builtin_amdgcn_ballot_w64(first || mx > PfSoftmax<DT>::kThreshold) != 0) {
            mx = fmaxf(mx, __shfl_xor(mx, 32));                  // the row's keys live in 2 lanes (h2)
            // The first keys a row sees put its reference kHeadroom above their maximum, wherever
            // that is (nothing has been accumulated yet); afterwards the reference only moves up
            // (rows with no visible key in the tile, or with lower scores, keep theirs).
            const bool sees = mx > -INFINITY;
            const float delta = first ? (sees ? mx + PfSoftmax<DT>::kHeadroom : 0.f)
                                      : fmaxf(mx + PfSoftmax<DT>::kHeadroom, 0.f);
            const float alpha = first ? 1.f : fast_exp2(-delta);
            started = started || sees;
            m_ref += delta;
            lsum *= alpha;
#pragma unroll
            for (int e = 0; e < 16; ++e) x[e] -= delta;
#pragma unroll
            for (int db = 0; db < kDB; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[db][e] *= alpha;
        }
        // weights as 2-byte pairs: pk[m] = B operand of the output MFMA over keys 16m .. 16m + 15
        // (its contraction slot (h2, e) is key 16m + 8(e / 4) + 4h2 + e % 4, elements 8m + e of x)
        uint32_t pk[2][4], pk_lo[2][4];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float w0 = fast_exp2(x[2 * e]), w1 = fast_exp2(x[2 * e + 1]);
            if (PfSoftmax<DT>::kSplitWeights) {
                split_bf16(w0, w1, pk[e >> 2][e & 3], pk_lo[e >> 2][e & 3]);
                lsum += w0 + w1;
            } else {
                // single rounding: normalise by the weights as rounded, so that the output stays
                // an exact convex combination of V rows
                const uint32_t hi = pack2<DT>(w0, w1);
                pk[e >> 2][e & 3] = hi;
                pk_lo[e >> 2][e & 3] = 0u;
                lsum += widen_lo<DT>(hi) + widen_hi<DT>(hi);
            }
        }

        // ---- O^T += V^T P^T ---------------------------------------------------------------------
        // A = V^T for dims 32db .. +31: this lane is dim 32db + n32 and needs keys 16m + 4h2 + (0..3)
        // and 16m + 8 + 4h2 + (0..3).  One transposing load hands each group of 16 lanes 4 keys x
        // 16 dims: lane s of a group addresses key (s / 4) of the four, dims 4 (s % 4) .. + 3.
        typedef short i16x4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) i16x4* lds_i16x4_ptr;
        const int s16 = lane & 15, dhalf = (lane >> 4) & 1;
        const uint16_t* vrow = &tile_lds[tile_base_v(buf) + (DIRECT ? Direct::keys_at(s16, dhalf, h2) / 2
                                                                    : (4 * h2 + (s16 >> 2)) * kPfVRow + 16 * dhalf + 4 * (s16 & 3))];
        auto further = [](int k8, int db) { return DIRECT ? Direct::further(k8, db) / 2 : 8 * k8 * kPfVRow + 32 * db; };
#pragma unroll
        for (int db = 0; db < kDB; ++db)
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)(vrow + further(2 * m, db)));
                const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_ptr)(vrow + further(2 * m + 1, db)));
                const uint2 lo2 = __builtin_bit_cast(uint2, lo), hi2 = __builtin_bit_cast(uint2, hi);
                const uint4 va = make_uint4(lo2.x, lo2.y, hi2.x, hi2.y);
                acc[db] = mfma32<DT>(va, make_uint4(pk[m][0], pk[m][1], pk[m][2], pk[m][3]), acc[db]);
                if (PfSoftmax<DT>::kSplitWeights)
                    acc[db] = mfma32<DT>(va, make_uint4(pk_lo[m][0], pk_lo[m][1], pk_lo[m][2], pk_lo[m][3]), acc[db]);
            }
    };

    // ---- the rest of the walk judged at once -------------------------------------------------------
    // 0 (for the whole workgroup) if no key of tiles 0 .. kt can carry a weight above 2^kPfSkipLog2 of
    // any row's sum so far - of the smaller of the two lanes' halves of it, which is what the test in softmax_pv
    // compares with - so that every one of these tiles would be skipped by that test anyway; else the number of
    // tiles after which it is worth asking again.  (A half below 2^-30 of the other counts as that much: where a row's
    // first visible keys are all one lane's, the other's half stays zero as long as its weights round to zero -
    // fp16, a steep slope, with two key groups 36 keys or more to the next of them - and a row without a sum wants
    // every tile.  What this leaves out is below 2^-54 of the row's sum a key.)
    // (A skipped tile still costs its fetch, score MFMAs and barrier, 0.45 us when tiles passed through registers; the keys read here
    // cost 0.1.  8 chunks of 512 behind 2 048, 32 / 8 heads: step 156 -> 120 us together with the rows by
    // head above; 8 prompts of 2 560: 452 -> 403.)
    // By Cauchy-Schwarz |q.k| <= |q||k|, so key j is out of the question for a row if
    //     |scale2| |q| |k_j| + slope2 * (j - pos) - m_ref  <=  log2(sum) + kPfSkipLog2,
    // i.e. |k_j| <= A + B * (k0 - j) with k0 the nearest of the keys, A = (log2(sum) + kPfSkipLog2 + m_ref
    // + slope2 * (pos - k0)) / (|scale2||q|), B = slope2 / (|scale2||q|) (any sign), the least A and B of
    // all rows.  The workgroup then reads the keys once, without V, LDS, MFMAs or exponentials.
    // A norm that is not a number, or infinite, fails the test.
    // When to ask: A grows by 32 B a tile, and the keys' norms - not known before they are read - are
    // taken to be like the queries', at most 1.25 |q| (a wrong guess costs time only).
    // A key that fails fails every later look too (but for the growth of the sum) until the walk is past it.  So a
    // look ends, for all waves, where the nearest failing key lies; the walk leaves out the tiles before it (restart)
    // and looks again behind it, when the bound has grown to the least norm of the key's group (all keys may be louder
    // than the queries) and after twice as many tiles each time (they may be loud here and there).  Chunks of 512
    // behind 32 000, 32 / 8 heads, one key of 10 times the norm at distance 2 000 / 20 000: 1 614 / 10 000 us when
    // every look read on past it and the next came 8 tiles later, 396 / 403 now, 718 without looks (none loud: 460, 387 and
    // 720); all of 10 times the norm: 1 396, 642 and 752.
    int pause = 2 * kPfCheckTiles, passed = 0;                   // passed: tiles kt, kt - 1, ... that a failing look has judged away
    auto rest_judged = [&](int kt) __attribute__((always_inline)) -> int {
        const int k0 = kt * kPfKeys + kPfKeys - 1;
        float q2 = 0.f;
#pragma unroll
        for (int m = 0; m < kQ; ++m) {
            q2 = dot2<DT>(qb[m].x, qb[m].x, q2);
            q2 = dot2<DT>(qb[m].y, qb[m].y, q2);
            q2 = dot2<DT>(qb[m].z, qb[m].z, q2);
            q2 = dot2<DT>(qb[m].w, qb[m].w, q2);
        }
        q2 += __shfl_xor(q2, 32);                                // a row's dims live in 2 lanes (h2)
        // (margins cover the rounding of the norms, 2^-58 the squares below 2^-126 that are lost in them: as many in the
        // keys' norms, which is why qs is bounded below)
        const float qn = __builtin_amdgcn_sqrtf(q2) + 0x1p-58f;
        const float qs = 1.001f * fabsf(scale2) * qn + 0x1p-100f;
        const float other = __shfl_xor(lsum, 32);
        const float half = row_ok ? fmaxf(fminf(lsum, other), 0x1p-30f * fmaxf(lsum, other)) : INFINITY;
        const float room = __builtin_amdgcn_logf(half) + (kPfSkipLog2 - 0.01f);
        float a = (room + m_ref + slope2 * (posf - (float)k0)) / qs;
        float bb = row_ok ? slope2 / qs : INFINITY;
        // (predicted from the whole sum first: near the diagonal one half may have hardly begun)
        const float ahead = row_ok ? (__builtin_amdgcn_logf(0.5f * (lsum + other)) - __builtin_amdgcn_logf(half)) / qs : 0.f;
        const float lack = 1.25f * qn - (a + ahead > 1.25f * qn ? a : a + ahead);
        float wait = lack <= 0.f ? 0.f : fminf(lack / (bb * (float)kPfKeys) + 1.f, 1e6f);
        wait = room == -INFINITY ? 1.f : wait >= 0.f ? wait : 1e6f;  // (no key seen yet; no slope, or a negative one)
        const bool no = !(a > 0.f && qs < 0x1p40f);
        if (__builtin_amdgcn_ballot_w64(no) != 0) a = -1.f;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            a = fminf(a, __shfl_xor(a, off));
            bb = fminf(bb, __shfl_xor(bb, off));
            wait = fmaxf(wait, __shfl_xor(wait, off));
        }
        if (lane == 0) {
            vote[0][wg_wave] = a;
            vote[1][wg_wave] = bb;
            vote[2][wg_wave] = wait;
            nearest_bad = -1;                                    // (the last call's have been read, barriers ago)
            least_norm2 = 0x7f800000u;
        }
        __syncthreads();
        a = vote[0][0], bb = vote[1][0], wait = vote[2][0];
#pragma unroll
        for (int i = 1; i < WAVES; ++i) {
            if (KS == 2 && i >= nwaves) break;
            a = fminf(a, vote[0][i]);
            bb = fminf(bb, vote[1][i]);
            wait = fmaxf(wait, vote[2][i]);
        }
        passed = 0;
        if (!(a > 0.f) || wait > 0.f) return max(kPfCheckTiles / 2, __builtin_amdgcn_readfirstlane((int)wait));    // workgroup-uniform
        // Nearest first, the waves take groups of 16 keys in turn: one block each, kLoads 16-byte loads per
        // lane, kRowLanes lanes to a key.  A lane holds the block number of one of the wave's next 64 groups.
        constexpr int kRowLanes = D * ES / 16, kRowsPerLoad = 64 / kRowLanes, kLoads = 16 / kRowsPerLoad;
        int s_lane = lane;
        asm volatile("" : "+v"(s_lane));                         // (keeps this rare code's addresses out of the registers of the loop around it)
        const int s_row = s_lane / kRowLanes, s_piece = s_lane % kRowLanes;
        const uint32_t row_bytes = CONTIG ? (uint32_t)(p.k_in_stride * 2) : D * ES;
        const int groups = (k0 + 1) / 16;
        const float far_end = bb < 0.f ? 15.f : 0.f;             // offset of a group's key with the least bound
        bool stop = false;                                       // wave-uniform
        for (int g0 = 0; g0 < groups && !stop; g0 += 64 * nwaves) {
            const int mine = min((groups - g0 - wg_wave + nwaves - 1) / nwaves, 64);     // this wave's groups here
            if (mine <= 0) break;
            auto base_key = [&](int i) __attribute__((always_inline)) { return k0 - 15 - 16 * (g0 + i * nwaves + wg_wave); };
            const int blks = CONTIG ? 0 : table[max(base_key(s_lane), 0) >> bs_shift];
            auto load_keys = [&](uint4 (&x)[kLoads], int i) __attribute__((always_inline)) {
                i = min(i, mine - 1);
                const int key = base_key(i);
                const int blk = CONTIG ? 0 : __builtin_amdgcn_readlane(blks, i);
                if (STEP && key + 15 >= pos0) {                  // some of its keys are new: from the inputs, chosen per key
#pragma unroll
                    for (int r = 0; r < kLoads; ++r) {
                        const int kk = key + kRowsPerLoad * r + s_row;
                        const unsigned char* src = kc + (uint64_t)(uint32_t)blk * l_blk_bytes + (uint32_t)((kk & (bs - 1)) * (D * ES));
                        if (kk >= pos0) src = kin + (uint64_t)(uint32_t)(kk - pos0) * (uint32_t)(p.k_in_stride * 2);
                        x[r] = *reinterpret_cast<const uint4*>(src + 16 * s_piece);
                    }
                    return;
                }
                const unsigned char* src = CONTIG ? kc + (uint64_t)(uint32_t)key * row_bytes
                                                  : kc + (uint64_t)(uint32_t)blk * l_blk_bytes + (uint32_t)((key & (bs - 1)) * (D * ES));
#pragma unroll
                for (int r = 0; r < kLoads; ++r)
                    x[r] = *reinterpret_cast<const uint4*>(src + (uint64_t)(uint32_t)(kRowsPerLoad * r + s_row) * row_bytes + 16 * s_piece);
            };
            auto norm2 = [&](uint4 y, float n2) __attribute__((always_inline)) {
                n2 = dot2<DT>(y.x, y.x, n2);
                n2 = dot2<DT>(y.y, y.y, n2);
                n2 = dot2<DT>(y.z, y.z, n2);
                return dot2<DT>(y.w, y.w, n2);
            };
            // (least: of the norms' squares)
            auto judge = [&](const uint4 (&x)[kLoads], int i, float& least) __attribute__((always_inline)) -> bool {
                const float most = fmaf(bb, (float)(k0 - 15 - base_key(min(i, mine - 1))) + far_end, a);
                const float most2 = most > 0.f ? fminf(most * most * 0.999f, 0x1p126f) : -1.f;
                bool bad = false;
                least = INFINITY;
#pragma unroll
                for (int r = 0; r < kLoads; ++r) {
                    float n2;
                    if constexpr (KV8) n2 = norm2(widen8_e4m3<DT>(x[r].z, x[r].w), norm2(widen8_e4m3<DT>(x[r].x, x[r].y), 0.f));
                    else n2 = norm2(x[r], 0.f);
                    n2 = row_group_sum<kRowLanes>(n2);
                    bad = bad || !(n2 <= most2);
                    least = fminf(least, n2);
                }
                return bad;
            };
            uint4 x0[kLoads], x1[kLoads];
            load_keys(x0, 0);
            for (int i = 0; i < mine && !stop; i += 2) {
                load_keys(x1, i + 1);
                const int others = *static_cast<volatile int*>(&nearest_bad);
                float least0, least1;
                const bool bad0 = judge(x0, i, least0);
                load_keys(x0, i + 2);
                const bool bad1 = judge(x1, i + 1, least1);
                if (__builtin_amdgcn_ballot_w64(bad0 || bad1) != 0) {
                    const bool first = __builtin_amdgcn_ballot_w64(bad0) != 0;
                    float least = first ? least0 : least1;
#pragma unroll
                    for (int off = kRowLanes; off < 64; off <<= 1) least = fminf(least, __shfl_xor(least, off));
                    if (lane == 0) {
                        atomicMax(&nearest_bad, base_key(first ? i : min(i + 1, mine - 1)));
                        atomicMin(&least_norm2, __builtin_bit_cast(uint32_t, least));
                    }
                    stop = true;
                }
                // (another wave's key that fails: nothing beyond it counts)
                stop = stop || __builtin_amdgcn_readfirstlane(others) > base_key(i);
            }
        }
        __syncthreads();
        const int nearest = __builtin_amdgcn_readfirstlane(nearest_bad);
        if (nearest < 0) return 0;
        const float quiet = __builtin_amdgcn_sqrtf(__builtin_bit_cast(float, least_norm2));
        const float grown = bb > 0.f ? fminf((quiet - a) / (bb * (float)kPfKeys) + 1.f, 1e6f) : 0.f;
        passed = kt - nearest / kPfKeys;
        const int next = max(passed + pause, __builtin_amdgcn_readfirstlane((int)grown));
        pause *= 2;
        return next;                                             // (the next call's votes are barriers away)
    };

    const int pos_min = pos0 + tq0;                             // tiles ending at or below it need no causal mask

    // Software pipeline: the score MFMAs of the walk's next tile are issued before the softmax of the
    // current one, so that the matrix pipe has work while the vector ALU does the exponentials
    // (measured: 3 % on the kernel).  For that the K tiles run one tile ahead of the V tiles: at the
    // start of step j, K tiles j and j + 1 and V tile j are in LDS, and K tile j + 2 and V tile j + 1 are
    // on their way to registers (DIRECT: are asked for now; DEEP: are on their way to LDS, and the ones
    // after them are asked for now).  Prologue:
    if constexpr (!DIRECT) {
        store_tile(stage_first, 0);
        if (k_loader) {                                          // wave-uniform
            store_tile(stage, 1);
            fetch_tile(stage, 2);
        }
    }
    if (own_tokens > 0) {                                        // the rows loaded at the top have landed with the tiles
        const global_byte_ptr cache = own_cache(threadIdx.x);
#pragma unroll
        for (int c = 0; c < kOwnBatch; ++c) {
            const int t = (int)threadIdx.x / (2 * kCPR) + c * own_step;
            int blk = own_blk[c];
            asm volatile("" : "+v"(blk));                        // (widened here and no earlier: at its load the widening waits for it)
            if (t < own_tokens) *own_dst(cache, t, blk) = own[c];
        }
    }
    __syncthreads();
    // the tiles that are on their way at the start of step j
    auto direct_lead = [&](int j) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 1; i < kLead; ++i)
            if (j + i + l_ahead < steps) direct_tile(j + i + l_ahead, std::false_type{});
    };
    direct_lead(0);
    f32x16 st_next = scores(0, [] {});
    __syncthreads();                                             // buffer 0's K tile may be overwritten during step 0
    // Tiles wholly inside every row's visible range need no mask: those that end at or below the
    // first row's position (causal side) and start at or above the last row's window start.
    const int n_unmasked = min(ntiles, max(0, (pos_min + 1) / kPfKeys));
    const int n_window_cut = W > 0 ? (max(kmax - W, 0) + kPfKeys - 1) / kPfKeys : 0;
    // (plain loops rather than one with a branch in it, and no branch around the stores: the
    // compiler schedules a loop whose body is one straight line far better)
    // While step j is computed, K tile j + 2 / V tile j + 1 (through registers: fetched one step earlier; DEEP: asked
    // for one step earlier, and the next ones are asked for) go into buffers that step j - 1 and those before it used;
    // the waves meet after every step.  (Two steps ahead is for walks that prefill_deep names, and never for whole
    // prompts: with a third buffer, 8 chunks of 512 behind 2 048 103.3 -> 107.2 us, 8 prompts of 2 560 350 -> 363.)
    // The last step's look-ahead scores read a stale K buffer and are never used; through registers, stores past
    // the last tile put the clamped re-read of it into a buffer nobody reads again, and DIRECT asks for none.
    // (two steps per trip with the two score registers swapping roles, so that no trip copies the
    // look-ahead scores into place)
    f32x16 st_other;
    auto one_tile = [&](int j, const f32x16& st_cur, f32x16& st_ahead, auto masked) __attribute__((always_inline)) {
        const bool more = j + kLead + l_ahead < steps;           // wave-uniform; nothing is asked for past the walk's end
        st_ahead = scores(j + 1, [&]() __attribute__((always_inline)) {
            if (DIRECT && more) direct_tile(j + kLead + l_ahead, std::false_type{});
        });
        softmax_pv(last_tile - ((j << share) + kw), j, st_cur, masked);
        if constexpr (DIRECT) {
            if (kLead == 1 || !more) wait_direct();
            else wait_direct<(kLead - 1) * kWaveGroups>();       // K tile j + 2 or V tile j + 1 is there, what was asked for later need not be
        } else {
            store_tile(stage, j + 1 + l_ahead);
            fetch_tile(stage, j + 2 + l_ahead);
        }
        __syncthreads();
    };
    // steps [from, to) of the walk
    auto run_tiles = [&](int from, int to, auto masked) __attribute__((always_inline)) {
        int j = from;
        // (as many steps to a trip as there are buffers, whose places are then the same in every trip)
        if constexpr (DEEP && !decltype(masked)::value && (!JUDGE || D == 64))
            for (; j + 3 < to; j += 4) {
                one_tile(j, st_next, st_other, masked);
                one_tile(j + 1, st_other, st_next, masked);
                one_tile(j + 2, st_next, st_other, masked);
                one_tile(j + 3, st_other, st_next, masked);
            }
        for (; j + 1 < to; j += 2) {
            one_tile(j, st_next, st_other, masked);
            one_tile(j + 1, st_other, st_next, masked);
        }
        if (j < to) {
            one_tile(j, st_next, st_other, masked);
            st_next = st_other;
        }
    };
    // The walk goes on at step j, wherever it was (every wave has passed a barrier since it last read a tile).
    auto restart = [&](int j) __attribute__((always_inline)) {
        if constexpr (DIRECT) {
            if constexpr (DEEP) wait_direct();                   // (tiles that are left out)
            direct_tile(j, std::false_type{});
            if (k_loader && j + 1 < steps) direct_tile(j + 1, std::false_type{});
            wait_direct();
        } else {
            blk_next = load_blk(j);
            fetch_tile(stage, j);
            store_tile(stage, j);
            if (k_loader) {
                fetch_tile(stage, j + 1);
                store_tile(stage, j + 1);
            }
            fetch_tile(stage, j + 1 + l_ahead);
        }
        __syncthreads();
        direct_lead(j);
        st_next = scores(j, [] {});
        __syncthreads();
    };
    const int cut_end = max(kt0, min(n_window_cut, n_unmasked));   // tiles cut by some row's window start
    const int plain_end = max(cut_end, n_unmasked);                // tiles no mask touches
    // from the diagonal backwards: the tiles the causal mask cuts come first, those that some
    // row's window start cuts (if there is a window) last
    // (in steps of a tile for each group: a step that any mask touches takes the masked path)
    const int from_plain = min((ntiles + pad - plain_end + share) >> share, steps);
    const int to_plain = WIN ? max(from_plain, ntiles - cut_end) : steps;
    run_tiles(0, from_plain, std::true_type{});
    // (Without slopes no weight is ever out of the question for its position alone: no JUDGE.)
    int ask = nt;
    for (int j = from_plain; j < to_plain;) {
        if constexpr (JUDGE)
            if (nt - (j << share) >= kPfJudgeTiles) {
                ask = rest_judged(last_tile - (j << share));
                if (ask == 0) break;
                if (passed >= kPfJumpTiles) {                    // workgroup-uniform
                    j += passed >> share;
                    ask -= passed >> share << share;
                    restart(j);
                }
            }
        const int to = min(j + ((ask + share) >> share), to_plain);
        run_tiles(j, to, std::false_type{});
        j = to;
    }
    if constexpr (WIN) run_tiles(to_plain, steps, std::true_type{});
    if constexpr (DEEP && JUDGE) {                               // tiles on their way that nobody reads any more: not into the output rows
        wait_direct();
        __syncthreads();
    }

    // ---- two key groups: merge (max / rescale / add), each wave of a pair finishing half of the dims ----
    // The waves of a row block hold the same rows in the same lanes; each leaves its reference, its sum
    // and the other's half of its output block in LDS, over the tile buffers.
    constexpr int kDBW = kDB / KS;                               // 32-dim blocks that this wave writes
    f32x16 (&res)[kDB] = acc;
    const int db0 = kw * kDBW;
    if constexpr (KS == 2) if (share) {
        constexpr int kPieces = kDBW * 4;                        // 16-byte pieces per lane and wave, and a pair of floats
        static_assert(DEEP ? WAVES * 64 * (kPieces * 16 + 8) == Direct::exchange_bytes(WAVES, KS)
                           : WAVES * 64 * (kPieces * 16 + 8) <= KS * PfTile<D>::kLdsBytes, "the exchange has its place");
        float4* const xch = reinterpret_cast<float4*>(tile_lds);
        float2* const xch_ml = reinterpret_cast<float2*>(xch + WAVES * 64 * kPieces);
        const int pair_mine = kw * kPfWaves + row_block, pair_theirs = (1 - kw) * kPfWaves + row_block;
        const int mine = pair_mine * kPieces * 64 + lane, theirs = pair_theirs * kPieces * 64 + lane;
        __syncthreads();
        const float m_mine = started ? m_ref : -INFINITY;        // (a group need not have seen a key of the row)
        xch_ml[pair_mine * 64 + lane] = make_float2(m_mine, lsum);
#pragma unroll
        for (int i = 0; i < kDBW; ++i) {
            const f32x16 send = kw == 0 ? acc[kDBW + i] : acc[i];
            if (kw != 0) res[i] = acc[kDBW + i];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                xch[mine + 64 * (4 * i + e)] = make_float4(send[4 * e], send[4 * e + 1], send[4 * e + 2], send[4 * e + 3]);
        }
        __syncthreads();
        const float2 t = xch_ml[pair_theirs * 64 + lane];
        const float m_all = fmaxf(m_mine, t.x);
        const float f0 = fast_exp2(m_mine - m_all), f1 = fast_exp2(t.x - m_all);
        lsum = lsum * f0 + t.y * f1;
#pragma unroll
        for (int i = 0; i < kDBW; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float4 o = xch[theirs + 64 * (4 * i + e)];
                res[i][4 * e] = fmaf(o.x, f1, res[i][4 * e] * f0);
                res[i][4 * e + 1] = fmaf(o.y, f1, res[i][4 * e + 1] * f0);
                res[i][4 * e + 2] = fmaf(o.z, f1, res[i][4 * e + 2] * f0);
                res[i][4 * e + 3] = fmaf(o.w, f1, res[i][4 * e + 3] * f0);
            }
    }

    // ---- normalise and write: this lane holds dims 32db + 8i + 4h2 + (0..3) of its row -----------
    unsigned char* const op = static_cast<unsigned char*>(p.out) + rows_base;
    float lt = lsum;
    lt += __shfl_xor(lt, 32);
    const float inv = out_scale / lt;
    // (addresses are worked out anew here: kept from the top, or this code moved into the walk's last trip, they would take
    // the walk's registers)
    int e_lane = lane;
    asm volatile("" : "+v"(e_lane));
    // dims 32 * block .. +31 of the lane's row, into the wave's strip
    auto put = [&](int block, const f32x16& x) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            u32x2 packed;
            packed.x = narrow2<DT>(x[4 * i] * inv, x[4 * i + 1] * inv);
            packed.y = narrow2<DT>(x[4 * i + 2] * inv, x[4 * i + 3] * inv);
            *reinterpret_cast<u32x2*>(strip + (e_lane & 31) * kPfKRow + 32 * block + 8 * i + 4 * (e_lane >> 5)) = packed;
        }
    };
    // the strip's rows that exist, pieces col0 .. col0 + PIECES - 1 of 16 bytes each
    auto write_rows = [&](auto pieces, int col0) __attribute__((always_inline)) {
        constexpr int PIECES = decltype(pieces)::value, kRows = 64 / PIECES;
        wave_lds_fence();
        const int piece = col0 + e_lane % PIECES;
#pragma unroll
        for (int m = 0; m < 32 / kRows; ++m) {
            const int r = kRows * m + e_lane / PIECES;
            const Row row = row_at(r);
            const u32x4 x = *reinterpret_cast<const u32x4*>(strip + r * kPfKRow + 8 * piece);
            if (row.ok) *reinterpret_cast<u32x4*>(op + row_offset(row) + 16 * piece) = x;
        }
    };
#pragma unroll
    for (int db = 0; db < kDBW; ++db) put(db0 + db, res[db]);
    if (KS == 2 && share) {
        write_rows(std::integral_constant<int, kCPR / KS>{}, db0 * 4);
    } else {                                                     // (alone: the other half as well)
#pragma unroll
        for (int db = kDBW; db < kDB; ++db) put(db, acc[db]);
        write_rows(std::integral_constant<int, kCPR>{}, 0);
    }
    // own rows beyond the first batch (stores inside the walk would delay the tile loads behind
    // them - loads and stores complete in issue order; measured twice as costly as this)
    if (own_tokens > kOwnBatch * own_step) {                     // workgroup-uniform
        int thread = threadIdx.x;
        asm volatile("" : "+v"(thread));
        const global_byte_ptr cache = own_cache(thread);
        for (int t = thread / (2 * kCPR) + kOwnBatch * own_step; t < own_tokens; t += own_step)
            *own_dst(cache, t, own_blk_of(t)) = *own_src(thread, t);
    }
}

// bytes of dynamic LDS
template <int D> constexpr int prefill_lds_bytes(int waves, int groups, bool deep)
{
    return deep ? PfDirect<D>::deep_lds_bytes(waves, groups) : PfTile<D>::lds_bytes(waves, groups);
}

template <int DT, bool KV8, bool WIN, bool CONTIG, bool JUDGE, int D, int WAVES, int KS, bool DEEP>
__global__ __launch_bounds__(WAVES * 64, OPTGQA_PF_WAVES_PER_SIMD) void paged_prefill_mma_kernel(const PrefillParams p)
{
    prefill_body<DT, KV8, WIN, CONTIG, JUDGE, D, WAVES, KS, DEEP, false>(p);
}

// cache write + prefill over the cached context in one launch (see STEP above)
template <int DT, bool JUDGE, int D, int WAVES, int KS, bool DEEP>
__global__ __launch_bounds__(WAVES * 64, OPTGQA_PF_WAVES_PER_SIMD) void paged_prefill_step_kernel(const PrefillParams p)
{
    prefill_body<DT, false, false, false, JUDGE, D, WAVES, KS, DEEP, true>(p);
}

}  // namespace optgqa
