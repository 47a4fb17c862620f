// KV-cache write and the un-paging diagnostic: pure index work and bit copies.
#pragma once
#include "common.hpp"
#include "optgqa.h"

namespace optgqa {

// Where a thread of the cache stores below works: 16-byte (or single-element) piece `piece` of one token, element off of its
// K and V rows.  A launch has fewer than 2^31 pieces (the host cuts longer ones by tokens), rows are a power of
// two of pieces and blocks of tokens: a multiplication and shifts.  (Divisions of 64-bit indexes, three a thread, were most of these
// kernels' time: 4 096 tokens of 8 heads of 128, 2-byte caches, 7.7 -> 6.7 us; 2 943 tokens into 8-bit
// caches 7.0 -> 5.4.)
struct CachePieces {
    FastDiv by_token;           // pieces of one token's K row
    int per_token, per_head_shift, num_pieces;      // pieces: of a token, of a head (log2), of all tokens
    int num_kv_heads, block_shift;
};

// What a cache store reads: the new tokens' rows, and where they go - their slots, or (a decode step) the block tables and
// lengths of the sequences.
struct StoreRows {
    const uint16_t *k, *v;
    int64_t k_stride, v_stride;         // elements from token to token
    const int64_t* slot_mapping;
    const int32_t *block_tables, *context_lens;     // (where slot_mapping is nullptr)
    int max_blocks_per_seq;

    // the same from token `first` on
    StoreRows from(int first) const
    {
        StoreRows s = *this;
        s.k += first * k_stride;
        s.v += first * v_stride;
        if (slot_mapping) {
            s.slot_mapping += first;
        } else {
            s.block_tables += (int64_t)first * max_blocks_per_seq;
            s.context_lens += first;
        }
        return s;
    }
};

// Launches of a cache store over slices of tokens of at most most_pieces pieces of `elems` elements each: one, but for K or V
// rows of 32 GiB (16-byte pieces) or 4 GiB (single elements).  call(rows of the slice, its pieces, its workgroups).
// Some 2^38 pieces and more are refused: 512 GiB of single elements, which no card holds, rows being a row apart at least.
template <typename F>
int for_cache_slices(const StoreRows& rows, int num_tokens, int num_kv_heads, int head_dim, int block_size, int elems, F&& call,
                     int most_pieces = 0x7fffffff)
{
    const int64_t per_token = (int64_t)num_kv_heads * (head_dim / elems);
    if (per_token > most_pieces || num_tokens * per_token > 128 * 0x7fffffffLL) return OPTGQA_ERR_SHAPE;
    CachePieces n;
    n.per_token = (int)per_token;
    n.by_token.set((uint32_t)per_token);
    n.per_head_shift = __builtin_ctz(head_dim / elems);
    n.num_kv_heads = num_kv_heads;
    n.block_shift = __builtin_ctz(block_size);
    const int most = (int)(most_pieces / per_token);        // tokens of a slice, >= 1
    for (int first = 0; first < num_tokens; ) {
        const int tokens = num_tokens - first < most ? num_tokens - first : most;
        n.num_pieces = (int)(tokens * per_token);
        const int rc = call(rows.from(first), n, dim3((unsigned)(((int64_t)n.num_pieces + 255) / 256)));
        if (rc != OPTGQA_OK) return rc;
        first += tokens;
    }
    return OPTGQA_OK;
}

// Cache store of Alg. 1 / eq. (2).  One thread moves one 16-byte piece (8 elements) of one
// token's K row and of its V row; pieces of a row are handled by consecutive lanes, so reads and
// writes are contiguous runs of head_dim * 2 bytes.  A padding token's rows are not read: they need not exist.
//   slot_mapping == nullptr (decode step): token t is the newest token of sequence t and goes to
//   position context_lens[t] - 1, whose slot is read from the block table; empty sequences skip.
template <typename VecT>
__global__ __launch_bounds__(256) void reshape_and_cache_kernel(
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v, uint16_t* __restrict__ k_cache,
    uint16_t* __restrict__ v_cache, const int64_t* __restrict__ slot_mapping, const CachePieces n,
    int64_t k_token_stride, int64_t v_token_stride,
    const int32_t* __restrict__ block_tables = nullptr, const int32_t* __restrict__ context_lens = nullptr,
    int max_blocks_per_seq = 0)
{
    constexpr int kElems = sizeof(VecT) / 2;
    const int64_t idx64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx64 >= n.num_pieces) return;
    const int idx = (int)idx64;
    const int t = n.by_token.div(idx), piece = idx - t * n.per_token;
    const int block_size = 1 << n.block_shift;
    int64_t block;
    int row;
    if (slot_mapping) {
        const int64_t slot = slot_mapping[t];
        if (slot < 0) return;                               // padding token
        block = slot >> n.block_shift;
        row = (int)slot & (block_size - 1);
    } else {
        const int pos = context_lens[t] - 1;
        if (pos < 0) return;
        block = block_tables[(int64_t)t * max_blocks_per_seq + (pos >> n.block_shift)];
        if (block < 0) return;                              // (no block: nothing to store to)
        row = pos & (block_size - 1);
    }
    const VecT kx = *reinterpret_cast<const VecT*>(k + t * k_token_stride + (int64_t)piece * kElems);
    const VecT vx = *reinterpret_cast<const VecT*>(v + t * v_token_stride + (int64_t)piece * kElems);
    const int g = piece >> n.per_head_shift, in_row = piece & ((1 << n.per_head_shift) - 1);
    const int64_t dst = ((((block * n.num_kv_heads + g) << n.block_shift) + row) << n.per_head_shift) * kElems + in_row * kElems;
    *reinterpret_cast<VecT*>(k_cache + dst) = kx;
    *reinterpret_cast<VecT*>(v_cache + dst) = vx;
}

// Cache store with a quantiser in front, for caches that hold 1-byte E4M3 codes (largest finite
// value 448, no infinities) and one scale per tensor, or - k_scales / v_scales given, device arrays
// of num_kv_heads values - one per KV head:
//     code = nearest_e4m3( fp32(x) * inv_scale ),  inv_scale = fp32(1 / scale): one correctly rounded
// fp32 division, on the host for the per-tensor scale, here for a KV head's.
// One fp32 multiplication, then e4m3_codes2 (round to nearest even, saturating, NaN -> 0x7f).
// One thread moves 8 elements of one token's K row and V row: 16 bytes in, 8 bytes out of each.
template <int DT>
__global__ __launch_bounds__(256) void reshape_and_cache_e4m3_kernel(
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v, unsigned char* __restrict__ k_cache,
    unsigned char* __restrict__ v_cache, const int64_t* __restrict__ slot_mapping, const CachePieces n,
    int64_t k_token_stride, int64_t v_token_stride,
    float k_inv_scale, float v_inv_scale, const float* __restrict__ k_scales, const float* __restrict__ v_scales)
{
    const int64_t idx64 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx64 >= n.num_pieces) return;
    const int idx = (int)idx64;
    const int t = n.by_token.div(idx), piece = idx - t * n.per_token;
    const int64_t slot = slot_mapping[t];
    if (slot < 0) return;                                   // padding token
    const uint4 kx = *reinterpret_cast<const uint4*>(k + t * k_token_stride + (int64_t)piece * 8);
    const uint4 vx = *reinterpret_cast<const uint4*>(v + t * v_token_stride + (int64_t)piece * 8);
    const int g = piece >> n.per_head_shift, in_row = piece & ((1 << n.per_head_shift) - 1);
    const int64_t row = slot & ((1 << n.block_shift) - 1);
    const int64_t dst = (((((slot >> n.block_shift) * n.num_kv_heads + g) << n.block_shift) + row) << n.per_head_shift) * 8 + in_row * 8;
    auto codes = [](const uint4& x, float inv) {
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
        uint32_t packed[2] = {0u, 0u};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t two = e4m3_codes2(widen_lo<DT>(w[i]) * inv, widen_hi<DT>(w[i]) * inv);
            packed[i >> 1] |= two << (16 * (i & 1));
        }
        return make_uint2(packed[0], packed[1]);
    };
    *reinterpret_cast<uint2*>(k_cache + dst) = codes(kx, k_scales ? 1.0f / k_scales[g] : k_inv_scale);
    *reinterpret_cast<uint2*>(v_cache + dst) = codes(vx, k_scales ? 1.0f / v_scales[g] : v_inv_scale);
}

// Un-paging: copy token j of sequence b, all KV heads, to dense [B][max_context_len][Hkv][D].
// One thread per 16-byte piece; grid = (ceil(max_context_len * pieces_per_token / 256), B, 2).
__global__ __launch_bounds__(256) void gather_kv_kernel(
    uint16_t* __restrict__ k_out, uint16_t* __restrict__ v_out, const uint16_t* __restrict__ k_cache,
    const uint16_t* __restrict__ v_cache, const int32_t* __restrict__ block_tables,
    const int32_t* __restrict__ context_lens, int num_kv_heads, int head_dim, int block_size,
    int max_blocks_per_seq, int max_context_len)
{
    const int b = blockIdx.y;
    const int pieces_per_head = head_dim / 8;
    const int pieces_per_token = num_kv_heads * pieces_per_head;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int j = (int)(idx / pieces_per_token);
    if (j >= context_lens[b] || j >= max_context_len) return;
    const int piece = (int)(idx - (int64_t)j * pieces_per_token);
    const int g = piece / pieces_per_head;
    const int d0 = (piece - g * pieces_per_head) * 8;
    const int64_t block = block_tables[(int64_t)b * max_blocks_per_seq + j / block_size];
    const int64_t src = ((block * num_kv_heads + g) * block_size + (j % block_size)) * head_dim + d0;
    const int64_t dst = (((int64_t)b * max_context_len + j) * num_kv_heads + g) * head_dim + d0;
    const uint16_t* cache = blockIdx.z == 0 ? k_cache : v_cache;
    uint16_t* out = blockIdx.z == 0 ? k_out : v_out;
    *reinterpret_cast<uint4*>(out + dst) = *reinterpret_cast<const uint4*>(cache + src);
}

}  // namespace optgqa
