// The library's host rules and index arithmetic, callable from the tests (tests/test_host_rules.py).
#include <setjmp.h>
#include <signal.h>
#include <stdlib.h>
#include <sys/mman.h>

#include <vector>

#include "cache_kernels.hpp"
#include "decode_kernels.hpp"
#include "decode_split.hpp"
#include "prefill_shape.hpp"

using namespace optgqa;

namespace {

sigjmp_buf out_of_range;
void on_fault(int) { siglongjmp(out_of_range, 1); }

// whether f touched nothing that is not mapped
template <typename F> bool in_range(F&& f)
{
    struct sigaction now = {}, before_segv, before_bus;
    now.sa_handler = on_fault;
    sigaction(SIGSEGV, &now, &before_segv);
    sigaction(SIGBUS, &now, &before_bus);
    const bool ok = sigsetjmp(out_of_range, 1) == 0;
    if (ok) f();
    sigaction(SIGSEGV, &before_segv, nullptr);
    sigaction(SIGBUS, &before_bus, nullptr);
    return ok;
}

// A copy of `bytes` bytes that ends where the mapped memory ends.
struct Guarded {
    char* base;
    size_t mapped, bytes;
    Guarded(const void* from, size_t n) : mapped((n + 4095) / 4096 * 4096), bytes(n)
    {
        base = static_cast<char*>(mmap(nullptr, mapped + 4096, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0));
        if (base == MAP_FAILED) abort();
        mprotect(base + mapped, 4096, PROT_NONE);
        memcpy(base + mapped - n, from, n);
    }
    ~Guarded() { munmap(base, mapped + 4096); }
    uint16_t* rows() const { return reinterpret_cast<uint16_t*>(base + mapped - bytes); }
};

template <typename F> void for_threads(dim3 grid, int threads, F&& f)
{
    blockDim = dim3(threads);
    for (blockIdx.x = 0; blockIdx.x < grid.x; ++blockIdx.x)
        for (threadIdx.x = 0; threadIdx.x < (uint32_t)threads; ++threadIdx.x) f();
}

}  // namespace

// The first of n numerators, by each divisor, whose quotient is not the processor's; -1: none.
extern "C" int64_t fast_div_differs(const uint32_t* divisors, int num_divisors, const int32_t* numerators, int n)
{
    for (int i = 0; i < num_divisors; ++i) {
        FastDiv d;
        d.set(divisors[i]);
        for (int j = 0; j < n; ++j)
            if ((uint32_t)d.div(numerators[j]) != (uint32_t)numerators[j] / divisors[i]) return (int64_t)i * n + j;
    }
    return -1;
}

// The same by an inverse that is `ulps` units in the last place off.
extern "C" int64_t div_by_inverse_differs(const int32_t* divisors, int num_divisors, const int32_t* numerators, int n, int ulps)
{
    for (int i = 0; i < num_divisors; ++i) {
        float inv = 1.0f / (float)divisors[i];
        for (int u = 0; u < abs(ulps); ++u) inv = nextafterf(inv, ulps > 0 ? INFINITY : 0.f);
        for (int j = 0; j < n; ++j)
            if (div_by_inverse(numerators[j], divisors[i], inv) != numerators[j] / divisors[i]) return (int64_t)i * n + j;
    }
    return -1;
}

// A cache store's launches in slices of at most most_pieces pieces, its kernel run thread by thread.  kind: 0 16-byte
// pieces, 1 single elements, 2 E4M3 codes (the low byte of the value, in place of the conversion).  rows: K and V rows that
// there are; reading others fails.  Returns the launches, -100 for a read or write out of range, or the refusal.
extern "C" int cache_store(int kind, const uint16_t* k, const uint16_t* v, int rows, int64_t k_stride, int64_t v_stride, void* k_cache, void* v_cache,
                           const int64_t* slots, const int32_t* tables, const int32_t* lens, int max_blocks, int tokens, int num_kv_heads,
                           int head_dim, int block_size, int most_pieces)
{
    const Guarded kg(k, 2 * rows * k_stride), vg(v, 2 * rows * v_stride);
    const StoreRows from{kg.rows(), vg.rows(), k_stride, v_stride, slots, tables, lens, max_blocks};
    int launches = 0, rc = 0;
    const bool ok = in_range([&] {
        rc = for_cache_slices(from, tokens, num_kv_heads, head_dim, block_size, kind == 1 ? 1 : 8, [&](const StoreRows& r, const CachePieces& n, dim3 grid) {
            ++launches;
            for_threads(grid, 256, [&] {
                auto kc = static_cast<uint16_t*>(k_cache);
                auto vc = static_cast<uint16_t*>(v_cache);
                if (kind == 2)
                    reshape_and_cache_e4m3_kernel<kBF16>(r.k, r.v, static_cast<unsigned char*>(k_cache), static_cast<unsigned char*>(v_cache),
                                                         r.slot_mapping, n, r.k_stride, r.v_stride, 1.f, 1.f, nullptr, nullptr);
                else if (kind == 1)
                    reshape_and_cache_kernel<uint16_t>(r.k, r.v, kc, vc, r.slot_mapping, n, r.k_stride, r.v_stride, r.block_tables, r.context_lens, r.max_blocks_per_seq);
                else
                    reshape_and_cache_kernel<uint4>(r.k, r.v, kc, vc, r.slot_mapping, n, r.k_stride, r.v_stride, r.block_tables, r.context_lens, r.max_blocks_per_seq);
            });
            return 0;
        }, most_pieces);
    });
    return !ok ? -100 : rc ? rc : launches;
}

// What for_cache_slices would launch (nothing is run): the slices' first tokens and pieces, up to `room` of them.
extern "C" int cache_slices(int64_t stride, int tokens, int num_kv_heads, int head_dim, int elems, int64_t* first, int64_t* pieces, int room)
{
    int n = 0;
    const uint16_t* const k = nullptr;
    const StoreRows from{k, k, stride, stride, nullptr, nullptr, nullptr, 1};
    const int rc = for_cache_slices(from, tokens, num_kv_heads, head_dim, 16, elems, [&](const StoreRows& r, const CachePieces& p, dim3 grid) {
        if (n == room || grid.x != (p.num_pieces + 255ll) / 256) return -99;
        first[n] = (int64_t)(reinterpret_cast<uintptr_t>(r.k) / 2) / stride;
        pieces[n++] = p.num_pieces;
        return 0;
    });
    return rc ? rc : n;
}

// An unsplit decode step's store of its new rows (every sequence's, KV head by KV head).
extern "C" int step_store(const uint16_t* k, const uint16_t* v, int rows, int64_t k_stride, int64_t v_stride, uint16_t* k_cache, uint16_t* v_cache,
                          const int32_t* tables, const int32_t* lens, int max_blocks, int num_seqs, int num_kv_heads, int head_dim, int block_size)
{
    const Guarded kg(k, 2 * rows * k_stride), vg(v, 2 * rows * v_stride);
    DecodeParams p = {};
    p.k_new = kg.rows(), p.v_new = vg.rows(), p.k_new_stride = k_stride, p.v_new_stride = v_stride;
    p.k_cache_w = k_cache, p.v_cache_w = v_cache;
    p.block_tables = tables, p.context_lens = lens, p.max_blocks_per_seq = max_blocks;
    p.num_seqs = num_seqs, p.num_kv_heads = num_kv_heads, p.block_size = block_size;
    return in_range([&] {
        for (int g = 0; g < num_kv_heads; ++g)
            for_threads(dim3(1), kDecodeWaves * 64, [&] { head_dim == 128 ? store_new_rows<128>(p, g) : store_new_rows<64>(p, g); });
    }) ? 1 : -100;
}

extern "C" int prefill_shape_of(int64_t units8, int shift, int max_q_len, int windowed, int cus)
{
    return (int)prefill_shape(units8, shift, max_q_len, windowed, cus);
}

extern "C" int prefill_shape_direct_of(int64_t units8, int shift, int max_q_len, int head_dim, int slopes, int windowed, int whole_prompts, int cus, int64_t key_bytes)
{
    return (int)prefill_shape_direct(units8, shift, max_q_len, head_dim, slopes, windowed, whole_prompts, cus, key_bytes);
}

extern "C" int prefill_deep_of(int64_t units8, int shift, int max_q_len, int slopes, int windowed, int cus, int64_t seen)
{
    return prefill_deep(units8, shift, max_q_len, slopes, windowed, cus, seen);
}

// The blocks that a wave would read, one after the other, through the numbers that its lanes hold (block n of the sequence: number
// n + 1000; read anew where they do not reach).  Returns the first that it would find wrong, or -1.
extern "C" int held_blocks_differ(const int32_t* blocks, int n, int* reads)
{
    int first = blocks[0], lanes[64];
    auto read = [&](int block) {
        first = block;
        for (int l = 0; l < 64; ++l) lanes[l] = (block - l > 0 ? block - l : 0) + 1000;
        ++*reads;
    };
    *reads = 0;
    read(first);
    for (int i = 0; i < n; ++i) {
        if (!held_blocks_reach(first, blocks[i])) read(blocks[i]);
        if (lanes[(first - blocks[i]) & 63] != blocks[i] + 1000) return i;
    }
    return -1;
}

extern "C" int decode_pairs_from_of(int64_t segments, int64_t rows, int max_context_len, int cus)
{
    return decode_pairs_from(segments, rows, max_context_len, cus);
}
