// Vector (non-MFMA) chunk kernels: Eq. (2b) restricted to the tokens of one chunk of one
// (sequence, selected KV head).  The path is HBM-bound (r flop per KV byte), so the layout
// is chosen for the loads, not for the ALUs:
//   - a (block, head) tile is 16 rows of D fp16 = 16*D*2 contiguous bytes; a wave reads
//     it with 128-bit loads, lane l taking bytes [16 l, 16 l + 16) of each 1 KB slice, so
//     D/8 neighbouring lanes hold one token row and a slice holds 64/(D/8) tokens;
//   - q.k is a v_dot2 chain per lane followed by a DPP sum over the D/8 lanes of a row;
//   - each group of D/8 lanes runs its own online softmax over the tokens it sees
//     (exp2 domain, fp32), so p never leaves registers between q.k and p.v;
//   - the lane groups of a wave are merged once per chunk, in a fixed order, by lane swaps.
// Nothing depends on how many heads were selected: the result for one (sequence, head)
// is a function of that sequence's length alone.
#pragma once
#include "attn_common.hpp"
#include "attn_persist.hpp"

namespace hetis {

template <int D, int R>
struct VecState {
    float m[R];
    float l[R];
    float o[R][8];

    __device__ __forceinline__ void reset()
    {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            m[r] = kNegBig;
            l[r] = 0.f;
#pragma unroll
            for (int x = 0; x < 8; ++x) o[r][x] = 0.f;
        }
    }
};

// Tiles are kept as vectors of words and taken apart by word: as a union of __half2 the compiler
// split the registers of a tile into halves right behind the load, for the next turn of the ring, and
// waited there for the loads it had just issued.  One tile pair was in flight instead of the ring (16
// chats x 13 heads of 128 29.1 -> 27.5 us, 640 rows of 7000 tokens 365 -> 353, 3072 rows of 1100 tokens
// of 64 dims 164 -> 150; 1664 rows of 1069 tokens, where memory is the bound either way, within 1 %).
template <int D>
struct TileRegs {
    static constexpr int NI = 16 / (512 / D);   // 1 KB slices per tile
    u32x4 k[NI];
    u32x4 v[NI];
};

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f16x2 as_f16x2(unsigned w) { return __builtin_bit_cast(f16x2, w); }

// One tile (16 tokens) of K and V held in registers -> update of the running state.  MASKED: only the
// first n_valid tokens count; the rows past them were loaded as zeros (see tile_rsrc), so their weight
// of zero meets no NaN.
template <int D, int R, bool MASKED>
__device__ __forceinline__ void vec_tile_update(VecState<D, R> &st, const TileRegs<D> &t,
                                                const f16x2 (&qh)[R][4], float scale_log2,
                                                int gid, int n_valid)
{
#pragma clang fp contract(off)
    // (every fused operation is written as one: two copies of this code must produce the same bits)
    constexpr int LPR = D / 8;        // lanes per token row
    constexpr int TPI = 64 / LPR;     // tokens per 1 KB slice
    constexpr int NI = 16 / TPI;      // slices per tile
    float s[NI][R];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const bool valid = !MASKED || (i * TPI + gid < n_valid);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float acc = 0.f;
#pragma unroll
            for (int x = 0; x < 4; ++x)
                acc = __builtin_amdgcn_fdot2(as_f16x2(t.k[i][x]), qh[r][x], acc, false);
            acc = group_sum<LPR>(acc);
            s[i][r] = valid ? acc * scale_log2 : -INFINITY;
        }
    }
    float p[NI][R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float mx = st.m[r];
#pragma unroll
        for (int i = 0; i < NI; ++i) mx = fmaxf(mx, s[i][r]);
        const float alpha = fast_exp2(st.m[r] - mx);
        st.m[r] = mx;
        float ps = 0.f;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            p[i][r] = fast_exp2(s[i][r] - mx);
            ps += p[i][r];
        }
        st.l[r] = __builtin_fmaf(st.l[r], alpha, ps);
#pragma unroll
        for (int x = 0; x < 8; ++x) st.o[r][x] *= alpha;
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const u32x4 vv = t.v[i];
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const float vf = (float)as_f16x2(vv[x / 2])[x % 2];
#pragma unroll
            for (int r = 0; r < R; ++r) st.o[r][x] = fmaf(p[i][r], vf, st.o[r][x]);
        }
    }
}

// Tile that may be the ragged last block of a sequence (n_valid < 16).
template <int D, int R>
__device__ __forceinline__ void vec_tile_update_any(VecState<D, R> &st, const TileRegs<D> &t,
                                                    const f16x2 (&qh)[R][4], float scale_log2,
                                                    int gid, int n_valid)
{
    if (n_valid < kBlockTokens)
        vec_tile_update<D, R, true>(st, t, qh, scale_log2, gid, n_valid);
    else
        vec_tile_update<D, R, false>(st, t, qh, scale_log2, gid, kBlockTokens);
}

// State of one piece into the state of the pieces before it, lane by lane (sums that are scaled in place: with
// the products the other way round every register took a move as well).
template <int D, int R>
__device__ __forceinline__ void vec_fold(VecState<D, R> &tot, const VecState<D, R> &st)
{
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma clang fp contract(off)
        const float M = fmaxf(tot.m[r], st.m[r]);
        const float a = fast_exp2(tot.m[r] - M), b = fast_exp2(st.m[r] - M);
        tot.m[r] = M;
        tot.l[r] = __builtin_fmaf(st.l[r], b, tot.l[r] * a);
#pragma unroll
        for (int x = 0; x < 8; ++x) tot.o[r][x] = __builtin_fmaf(st.o[r][x], b, tot.o[r][x] * a);
    }
}

// Merge the 64/(D/8) lane groups of a wave, neighbours first; the first group ends up with the sum.
template <int D, int R>
__device__ __forceinline__ void vec_wave_merge(VecState<D, R> &st)
{
#pragma clang fp contract(off)
    auto merge = [&](auto pair) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const LanePair m = pair(st.m[r]), l = pair(st.l[r]);
            const float M = fmaxf(m.lo, m.hi);
            const float a = fast_exp2(m.lo - M), b = fast_exp2(m.hi - M);
            st.m[r] = M;
            st.l[r] = __builtin_fmaf(l.lo, a, l.hi * b);
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const LanePair o = pair(st.o[r][x]);
                st.o[r][x] = __builtin_fmaf(o.lo, a, o.hi * b);
            }
        }
    };
    if constexpr (D == 64) merge([](float x) { return LanePair{x, dpp_mov<0x128>(x)}; });   // row_ror 8
    merge([](float x) { return pair_xor16(x); });
    merge([](float x) { return pair_xor32(x); });
}

// ---------------------------------------------------------------------------------------
// Policy through which the persistent kernel (attn_persist.hpp) uses the vector arithmetic.
// ---------------------------------------------------------------------------------------
template <int D_, int R_>
struct VecPolicy {
    static constexpr int D = D_;
    static constexpr int R = R_;
    static constexpr int kWaveLdsBytes = 0;      // no per-wave staging area
    static constexpr int kWavesPerEu = 2;        // register budget: 512 / 2 per lane
    // Tile pairs in flight per wave: 8 KB (a tile pair is 8 KB at D = 128, 4 KB at 64) in decode calls of
    // many rows, 16 KB (`deep`) in those of few or of short rows (deep_ring()) and in split calls.  8 KB in
    // each of 1024 waves already keep HBM busy (random 4 KB tiles: 6.85 TB/s with one, two or three pairs a
    // wave); more of it only waits longer, and not equally long on all compute units, which shows at the
    // end of a launch: with 16 and 8 KB 1664 rows of 1069 tokens 147.4 and 145.0 us (behind a block table
    // of 32k tokens 148.1 and 146.3), 1024 rows of 1088 97.6 and 96.7, 1600 rows of 900 (r = 2) 126 and
    // 124, 640 rows of 7000 353 and 350.  Where waves run dry before the launch ends those at work need
    // more each: 16 chats x 13 heads 27.9 us with 8 KB and 27.5 with 16, two documents x 8 heads 45.0 and
    // 40.8, 440 rows of 1250 tokens 57.6 and 55.0.  Split calls have no segments to even out and gain as
    // well (320 long rows 546 and 537).
    static constexpr int ring(bool deep) { return (deep ? 2 : 1) * (D_ == 64 ? 2 : 1); }
    // of a team's wave, whose piece is four tiles: a second turn costs less than twice the code (4: 32 rows of 600
    // tokens 11.0 -> 11.5, 16 of 2000 10.7 -> 11.2)
    static constexpr int kTeamRing = 2;
    static constexpr int ring_split = ring(true);
    using Tile = TileRegs<D>;
    using State = VecState<D, R>;
    struct Query {
        f16x2 h[R][4];                           // this lane's 8 dims of each head of the group
    };

    // K and V: lane l takes bytes [16 l, 16 l + 16) of every 1 KB slice of the tile
    __device__ static __forceinline__ void issue(Tile &t, __amdgpu_buffer_rsrc_t rk,
                                                 __amdgpu_buffer_rsrc_t rv, int lane)
    {
        const int voff = lane * 16;
#pragma unroll
        for (int i = 0; i < Tile::NI; ++i) t.k[i] = buffer_load_u4(rk, voff + i * 1024);
#pragma unroll
        for (int i = 0; i < Tile::NI; ++i) t.v[i] = buffer_load_u4(rv, voff + i * 1024);
    }
    using QueryPrefetch = Query;                 // loaded from global in its final layout
    __device__ static __forceinline__ void q_prefetch(QueryPrefetch &q, const __half *rows, int lane)
    {
        const int sub = lane % (D / 8);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const u32x4 t = *reinterpret_cast<const u32x4 *>(rows + r * D + sub * 8);
#pragma unroll
            for (int x = 0; x < 4; ++x) q.h[r][x] = as_f16x2(t[x]);
        }
    }
    __device__ static __forceinline__ void q_commit(Query &q, const QueryPrefetch &pre,
                                                    unsigned char *, int)
    {
        q = pre;
    }
    __device__ static __forceinline__ void reset(State &st) { st.reset(); }
    // MAYBE_RAGGED: the tile may be the ragged last block of a sequence (n_valid < 16); a
    // separate masked copy of the arithmetic keeps whole tiles free of compares and selects
    // kOneCopy: the masked copy for all tiles, where fetching the code costs more than the selects
    template <int MAYBE_RAGGED>
    __device__ static __forceinline__ void update(State &st, const Tile &t, const Query &q,
                                                  float scale_log2, int lane, int n_valid)
    {
        if (MAYBE_RAGGED == kOneCopy)
            vec_tile_update<D, R, true>(st, t, q.h, scale_log2, lane / (D / 8), n_valid);
        else if (MAYBE_RAGGED)
            vec_tile_update_any<D, R>(st, t, q.h, scale_log2, lane / (D / 8), n_valid);
        else
            vec_tile_update<D, R, false>(st, t, q.h, scale_log2, lane / (D / 8), kBlockTokens);
    }
    __device__ static __forceinline__ void fold(State &tot, const State &st) { vec_fold<D, R>(tot, st); }
    // The sums as they stand, in registers: no arithmetic on them moves past this point.
    __device__ static __forceinline__ void settle(State &st)
    {
#pragma unroll
        for (int r = 0; r < R; ++r)
            asm volatile("" : "+v"(st.m[r]), "+v"(st.l[r]), "+v"(st.o[r][0]), "+v"(st.o[r][1]), "+v"(st.o[r][2]),
                         "+v"(st.o[r][3]), "+v"(st.o[r][4]), "+v"(st.o[r][5]), "+v"(st.o[r][6]), "+v"(st.o[r][7]));
    }
    // state <-> LDS, sixteen bytes a lane at a time
    static_assert(R <= 2, "maximum and sum of all rows in one vector");
    static constexpr int kStateVecs = 2 * R + 1;
    __device__ static __forceinline__ void deposit(const State &st, f32x4 *to, int lane)
    {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            to[2 * r * 64 + lane] = f32x4{st.o[r][0], st.o[r][1], st.o[r][2], st.o[r][3]};
            to[(2 * r + 1) * 64 + lane] = f32x4{st.o[r][4], st.o[r][5], st.o[r][6], st.o[r][7]};
        }
        to[2 * R * 64 + lane] = f32x4{st.m[0], st.l[0], st.m[R - 1], st.l[R - 1]};
    }
    __device__ static __forceinline__ void collect(State &st, const f32x4 *from, int lane)
    {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const f32x4 lo = from[2 * r * 64 + lane], hi = from[(2 * r + 1) * 64 + lane];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                st.o[r][x] = lo[x];
                st.o[r][4 + x] = hi[x];
            }
        }
        const f32x4 ml = from[2 * R * 64 + lane];
        st.m[0] = ml[0];
        st.l[0] = ml[1];
        st.m[R - 1] = ml[2 * (R - 1)];
        st.l[R - 1] = ml[2 * (R - 1) + 1];
    }
    // normalised rows and their base-2 log-sum-exp -> LDS (the wave's mailbox)
    __device__ static __forceinline__ void finish(State &st, float (&o)[R][D], float (&lse)[R],
                                                  int lane)
    {
        vec_wave_merge<D, R>(st);                // the first lane group now holds the totals
        const int gid = lane / (D / 8), sub = lane % (D / 8);
        if (gid == 0) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float inv = __builtin_amdgcn_rcpf(st.l[r]);
                float4 lo = make_float4(st.o[r][0] * inv, st.o[r][1] * inv, st.o[r][2] * inv,
                                        st.o[r][3] * inv);
                float4 hi = make_float4(st.o[r][4] * inv, st.o[r][5] * inv, st.o[r][6] * inv,
                                        st.o[r][7] * inv);
                *reinterpret_cast<float4 *>(&o[r][sub * 8]) = lo;
                *reinterpret_cast<float4 *>(&o[r][sub * 8 + 4]) = hi;
                if (sub == 0) lse[r] = st.m[r] + fast_log2(st.l[r]);
            }
        }
    }
};

// Log-sum-exp merge of the partial results of a row's segments: one workgroup of D threads per
// (sequence, selected query row); in pairs mode per (pair, row of the group).  Bound by latency (a
// row's partial results are a few KB), so what counts is the chain of loads: the log-sum-exps of
// 64 segments take one load, a lane each, and their weights one exponential a lane; the partial
// results of kMergeBatch segments are in flight at the same time as the log-sum-exps, which they do
// not depend on.  The sums keep their order: ascending segments.
// This launch alone, against one load of each kind after the other: 8 x 40 rows of up to 32 segments
// 4.7 -> 4.0 us, 200 x 8 of 17 to 33 10.8 -> 7.3, 64 x 13 of up to 4 3.1 -> 2.8, 8 rows of up to 250
// 10.1 -> 10.3.
constexpr int kMergeBatch = 32;
template <int D>
__global__ __launch_bounds__(D) void attn_merge_kernel(const AttnParams p, int group)
{
    const int j = blockIdx.x;            // selected row: i*group + rr
    const int b = blockIdx.y;
    const int d = threadIdx.x, lane = threadIdx.x & 63;
    const bool pairs = p.pair_seq != nullptr;
    const int seq = pairs ? p.pair_seq[b] : b;
    const int n_sel = pairs ? 1 : p.n_sel;
    const int head = pairs ? p.pair_head[b] : p.head_ids[j / group];
    const int L = p.seq_lens[seq];
    const int n_segs = (L + p.seg_tokens - 1) / p.seg_tokens;
    if (p.direct_single && n_segs <= 1) return;        // already written by the chunk kernel
    __half *o = p.out + ((int64_t)seq * p.n_q_heads + head * group + j % group) * D;
    if (n_segs <= 0) {
        o[d] = __float2half_rn(0.f);
        return;
    }
    // partial of segment c of this row: index ((b*n_sel + i)*max_segs + c)*group + rr
    const int64_t base = ((int64_t)b * n_sel + j / group) * p.max_segs * group + j % group;
    const float *lse = p.lse_partial + base;
    const float *op = p.o_partial + base * D + d;
    float W = 0.f, acc = 0.f;
    if (n_segs <= 4) {
        // nothing to share between lanes (a split call over 6600 rows of one segment: 83.1 us without
        // this branch, 81.6 with it)
        float lc[4], x4[4], M = -INFINITY;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u >= n_segs) break;
            lc[u] = lse[(int64_t)u * group];
            x4[u] = op[(int64_t)u * group * D];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (u < n_segs) M = fmaxf(M, lc[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (u >= n_segs) break;
            const float w = fast_exp2((lc[u] - M) * kLog2e);
            W += w;
            acc = fmaf(w, x4[u], acc);
        }
        o[d] = __float2half_rn(acc / W);
        return;
    }
    auto lse_of = [&](int c) { return lse[(int64_t)min(c, n_segs - 1) * group]; };
    float x[kMergeBatch], next[kMergeBatch];
    auto load_batch = [&](float (&to)[kMergeBatch], int c0) {
#pragma unroll
        for (int g = 0; g < kMergeBatch; g += 8) {
            if (c0 + g >= n_segs) break;               // rows of few segments: no loads for nothing
#pragma unroll
            for (int u = g; u < g + 8; ++u) to[u] = op[(int64_t)min(c0 + u, n_segs - 1) * group * D];
        }
    };
    float l = lse_of(lane);                            // lane: segment c0 + lane of the group of 64
    load_batch(x, 0);
    float M = l;
#pragma unroll 4
    for (int c0 = 64; c0 < n_segs; c0 += 64) M = fmaxf(M, lse_of(c0 + lane));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, 64));
    int w_lane = 0;
    auto add = [&](int u, int c) {
        const float w = __int_as_float(__builtin_amdgcn_readlane(w_lane, c & 63));
        W += w;
        acc = fmaf(w, x[u], acc);
    };
#pragma unroll 1
    for (int c0 = 0; c0 < n_segs; c0 += kMergeBatch) {
        if (c0 % 64 == 0) {
            w_lane = __float_as_int(fast_exp2((l - M) * kLog2e));
            l = lse_of(c0 + 64 + lane);
        }
        if (c0 + kMergeBatch >= n_segs) {
#pragma unroll
            for (int u = 0; u < kMergeBatch; ++u) {
                if (c0 + u >= n_segs) break;
                add(u, c0 + u);
            }
            break;
        }
        load_batch(next, c0 + kMergeBatch);
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) add(u, c0 + u);
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) x[u] = next[u];
    }
    o[d] = __float2half_rn(acc / W);
}

}  // namespace hetis
