// Head-wise cache management kernels (Section 6, "KV cache management"): rows addressed by
// (sequence id, position, head id) through the block table, and whole (block, head) tiles
// copied between pools.  Pure data movement in 16-byte pieces; every index read from device
// memory is range-checked and an entry that fails the check is skipped.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hetis {

typedef unsigned int kv_u32x4 __attribute__((ext_vector_type(4)));

constexpr int kKvBlockTokens = 16;

struct KvRowParams {
    uint4 *rows_k;              // STORE: source rows [n_tokens, Hkv, D]; FETCH: destination
    uint4 *rows_v;
    uint4 *cache_k;             // STORE: destination; FETCH: source
    uint4 *cache_v;
    const int32_t *token_seq;   // or nullptr: entry n belongs to sequence n
    const int32_t *token_pos;   // position = token_pos[n] + pos_bias
    const int32_t *block_table;
    const int32_t *head_ids;
    int64_t stride_block, stride_head;   // in 16-byte units
    int64_t num_blocks;
    int32_t n_tokens, n_sel, n_kv_heads, batch, max_blocks_per_seq, pos_bias;
};

// One workgroup moves the K and V rows of kKvRowsPerWg<D> consecutive entries and ONE selected
// head: D/8 lanes per entry, 16 bytes of K and 16 bytes of V a lane.  Workgroups are numbered
// heads fastest, so that those that run at the same time cover a compact piece of both sides.
// HBM-bound.  How much of the copy a workgroup holds decides the rate: reads and writes mixed
// over a small window of addresses run faster than many streams far apart, so a thread does one
// access per operand and the grid is as large as the work, instead of a loop over the heads with
// eight rows in flight (one prompt store of 34k tokens x 13 heads x 128: 93.7 -> 87.3 us, the
// fetch of the same rows 92.3 -> 82.4; 1 GiB copied the same way without an index: 6.3 TB/s).  K
// and V by the same thread, because the index loads ahead of the first access are a chain of
// two memory latencies: with one 16-byte access a thread the same launches take 103 us.
constexpr int kKvRowThreads = 256;
template <int D>
constexpr int kKvRowsPerWg = kKvRowThreads / (D / 8);

template <int D, bool FETCH>
__device__ __forceinline__ void move_rows(const KvRowParams &p, int64_t n, int s, int c)
{
    constexpr int LR = D / 8;                   // lanes per row
    const int g = p.head_ids[s];
    const int64_t b = p.token_seq ? (int64_t)p.token_seq[n] : n;
    const int64_t pos = (int64_t)p.token_pos[n] + p.pos_bias;
    if (g < 0 || g >= p.n_kv_heads || b < 0 || b >= p.batch || pos < 0) return;
    const int64_t j = pos / kKvBlockTokens;
    if (j >= p.max_blocks_per_seq) return;
    const int64_t blk = p.block_table[b * p.max_blocks_per_seq + j];
    if (blk < 0 || blk >= p.num_blocks) return;
    const int64_t cache_row = blk * p.stride_block + g * p.stride_head + (pos % kKvBlockTokens) * LR + c;
    const int64_t rows_row = (n * p.n_kv_heads + g) * LR + c;
    const uint4 *src_k = FETCH ? p.cache_k + cache_row : p.rows_k + rows_row;
    const uint4 *src_v = FETCH ? p.cache_v + cache_row : p.rows_v + rows_row;
    uint4 *dst_k = FETCH ? p.rows_k + rows_row : p.cache_k + cache_row;
    uint4 *dst_v = FETCH ? p.rows_v + rows_row : p.cache_v + cache_row;
    // every byte is touched once: non-temporal both ways
    const kv_u32x4 k = __builtin_nontemporal_load((const kv_u32x4 *)src_k);
    const kv_u32x4 v = __builtin_nontemporal_load((const kv_u32x4 *)src_v);
    __builtin_nontemporal_store(k, (kv_u32x4 *)dst_k);
    __builtin_nontemporal_store(v, (kv_u32x4 *)dst_v);
}

// x: selected heads, y: groups of entries; a grid that does not reach strides on.
template <int D, bool FETCH>
__global__ void __launch_bounds__(kKvRowThreads) kv_rows_kernel(KvRowParams p)
{
    constexpr int LR = D / 8;
    constexpr int64_t N = kKvRowsPerWg<D>;
    for (int64_t n0 = blockIdx.y * N; n0 < p.n_tokens; n0 += gridDim.y * N) {
        const int64_t n = n0 + threadIdx.x / LR;
        if (n >= p.n_tokens) continue;
        for (int64_t s = blockIdx.x; s < p.n_sel; s += gridDim.x)
            move_rows<D, FETCH>(p, n, (int)s, threadIdx.x % LR);
    }
}

struct KvPairParams {
    const uint4 *k_new, *v_new;     // [batch, Hkv, D]
    uint4 *k_tiles, *v_tiles;       // single-head tiles
    const int32_t *block_table;     // [n_pairs, max_blocks_per_seq]
    const int32_t *seq_lens, *pair_seq, *pair_head;
    int64_t stride_tile;            // in 16-byte units
    int64_t num_tiles;
    int32_t n_pairs, n_kv_heads, batch, max_blocks_per_seq;
};

// Decode-step store for per-request head subsets: 2*D/8 lanes move the new K row and V row
// of one (sequence, KV head) pair to position seq_lens[b] - 1 through the pair's own
// block-table row.  Same checks as kv_rows_kernel; a pair that fails one is skipped.
template <int D>
__global__ void __launch_bounds__(256) kv_append_pairs_kernel(KvPairParams p)
{
    constexpr int LR = D / 8;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t pr = t / (2 * LR);
    if (pr >= p.n_pairs) return;
    const int within = (int)(t % (2 * LR));
    const bool is_v = within >= LR;
    const int c = within % LR;
    const int64_t b = p.pair_seq[pr];
    const int64_t g = p.pair_head[pr];
    if (b < 0 || b >= p.batch || g < 0 || g >= p.n_kv_heads) return;
    const int64_t pos = (int64_t)p.seq_lens[b] - 1;
    if (pos < 0) return;
    const int64_t j = pos / kKvBlockTokens;
    if (j >= p.max_blocks_per_seq) return;
    const int64_t tile = p.block_table[pr * p.max_blocks_per_seq + j];
    if (tile < 0 || tile >= p.num_tiles) return;
    const uint4 *src = (is_v ? p.v_new : p.k_new) + (b * p.n_kv_heads + g) * LR + c;
    uint4 *dst = (is_v ? p.v_tiles : p.k_tiles) + tile * p.stride_tile + (pos % kKvBlockTokens) * LR + c;
    *dst = *src;
}

struct KvCopyParams {
    const uint4 *src_k, *src_v;
    uint4 *dst_k, *dst_v;
    const int32_t *src_blocks, *dst_blocks, *src_heads, *dst_heads;
    int64_t src_stride_block, src_stride_head, dst_stride_block, dst_stride_head;   // 16-byte units
    int64_t src_num_blocks, dst_num_blocks;
    int32_t n_sel, src_n_heads, dst_n_heads;
};

// Tiles in the order pair, head, K before V; one 16-byte access a thread, so a workgroup moves
// one tile at D = 128 and two at D = 64, and a wave is always inside one tile (its indices are
// scalar).  HBM-bound.  As with the rows above the grid is as large as the work: 900 MB of tiles
// (64 prompts, 13 heads of 128) take 169.7 us this way, 5.4 TB/s read + written, and took 184.8 us
// with 2048 resident workgroups that strode over the tiles with 8 KB in flight per wave.  Loads
// and stores are non-temporal: every byte is touched once (cached stores 179 us, cached both ways
// 186 us).  K and V by the same thread: 180 us.  No loop around the body: with one the compiler
// fetches the indices by vector loads, because a store may precede them (208 us).  The price is more
// workgroups to start: copies of 1400 to 10 000 tiles of 2 KB (D = 64) take 0.1 to 0.6 us longer than
// with the resident ones (2000 pairs, one head: 5.0 -> 5.5 us), larger and smaller ones less.
constexpr int kKvCopyThreads = 256;

template <int D>
__global__ void __launch_bounds__(kKvCopyThreads) kv_copy_tiles_kernel(KvCopyParams p)
{
    constexpr int TV = kKvBlockTokens * D / 8;            // 16-byte units per tile
    constexpr int TILES = kKvCopyThreads / TV;            // tiles per workgroup
    const int in_wg = __builtin_amdgcn_readfirstlane((int)threadIdx.x / TV);
    const int unit = threadIdx.x % TV;
    const int t = blockIdx.x * TILES + in_wg, s = t >> 1, i = blockIdx.y;
    if (s >= p.n_sel) return;
    const int64_t sb = p.src_blocks[i], db = p.dst_blocks[i];
    const int sg = p.src_heads[s], dg = p.dst_heads[s];
    if (sb < 0 || sb >= p.src_num_blocks || db < 0 || db >= p.dst_num_blocks) return;
    if (sg < 0 || sg >= p.src_n_heads || dg < 0 || dg >= p.dst_n_heads) return;
    const uint4 *src = (t & 1) ? p.src_v : p.src_k;
    uint4 *dst = (t & 1) ? p.dst_v : p.dst_k;
    src += sb * p.src_stride_block + sg * p.src_stride_head + unit;
    dst += db * p.dst_stride_block + dg * p.dst_stride_head + unit;
    __builtin_nontemporal_store(__builtin_nontemporal_load((const kv_u32x4 *)src), (kv_u32x4 *)dst);
}

}  // namespace hetis
