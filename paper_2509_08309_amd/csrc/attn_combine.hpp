// What the two ways through the Attention kernel share: the cut of a row into chunks, the scans of the
// enumeration, the fold of chunk results and its stores, waits on words in LDS.
#pragma once
#include "attn_common.hpp"

namespace hetis {

enum : int { kMailEmpty = 0, kMailFull = 1, kMailDone = 2 };
enum : int { kKindOut = 0, kKindPartial = 1, kKindZero = 2, kKindFold = 3 };
constexpr int kMaxQuickRows = 512;      // rows of a launch that may be handed out by single chunks
// Segments of at most 1/HETIS_FINE_CHUNK_BELOW of a whole one are cut into chunks of half the
// size, those of at most a quarter of that into chunks of a quarter of the size.
#ifndef HETIS_FINE_CHUNK_BELOW
#define HETIS_FINE_CHUNK_BELOW 4
#endif
static_assert(HETIS_FINE_CHUNK_BELOW >= 4, "a segment in quarter chunks is one item of a team");
// Between two looks of a wait, in units of 64 cycles.  The looks are few (five waves a compute unit); with
// four units in the writer wave and two in the others 4 chats x 4 heads of 64 dims take 9.7 us
// instead of 9.4, 15 rows of at most 96 tokens 9.3 instead of 9.1, launches of many rows the same.
constexpr int kPollSleep = 1;
// Looks before a wait gives up: 2^30 cycles of sleep, 0.4 s.  The longest real wait is for a chunk of the
// wave's own workgroup, 1024 tokens at most, some tens of microseconds.
constexpr int kSpinLimit = (1 << 24) / kPollSleep;
template <int N>
struct IntTag {
    static constexpr int value = N;
};

// Inclusive scans over the 64 lanes of a wave (DPP, no LDS traffic): sums, and maxima of x >= 0.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_or_zero(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xF, true);
}
__device__ __forceinline__ int wave_scan_sum(int x)
{
    x += dpp_or_zero<0x111, 0xF>(x);    // row_shr 1, 2, 4, 8: inside each row of 16 lanes
    x += dpp_or_zero<0x112, 0xF>(x);
    x += dpp_or_zero<0x114, 0xF>(x);
    x += dpp_or_zero<0x118, 0xF>(x);
    x += dpp_or_zero<0x142, 0xA>(x);    // row_bcast 15: into rows 1 and 3
    x += dpp_or_zero<0x143, 0xC>(x);    // row_bcast 31: into rows 2 and 3
    return x;
}
__device__ __forceinline__ int wave_max(int x)
{
    x = max(x, dpp_or_zero<0x111, 0xF>(x));
    x = max(x, dpp_or_zero<0x112, 0xF>(x));
    x = max(x, dpp_or_zero<0x114, 0xF>(x));
    x = max(x, dpp_or_zero<0x118, 0xF>(x));
    x = max(x, dpp_or_zero<0x142, 0xA>(x));
    x = max(x, dpp_or_zero<0x143, 0xC>(x));
    return __builtin_amdgcn_readlane(x, 63);
}

// A value that is the same in all lanes, visibly so: an operand of a load that the compiler takes to be
// lane-dependent, where the load needs a scalar, becomes a loop over the lanes (8 rows of 500 to 1500 tokens,
// r = 8, 15.5 -> 15.2 us; the combination of words, r < 4, has no such operands, and is slower with these).
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int64_t uniform(int64_t x)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// x / d for x >= 0, d > 0 the same in all lanes: integer division has no instruction of its
// own and costs about forty; the divisors of the enumeration are powers of two unless a caller
// of the split entry points chooses otherwise.
__device__ __forceinline__ int udiv(int x, int d)
{
    if (__builtin_expect((d & (d - 1)) == 0, 1)) return x >> __builtin_ctz(d);
    return x / d;
}

// Tokens per chunk of a segment of n_tok tokens: the shorter the segment, the later it is
// handed out and the finer it is cut, so that the chunks still running when the work runs out
// are short ones.  A function of the row's length and of constants only, like everything that
// shapes the arithmetic.
__device__ __forceinline__ int chunk_tokens_of(int n_tok, int chunk_tokens, int seg_tokens)
{
    int ct = chunk_tokens;
    if (seg_tokens > chunk_tokens) {
        if (n_tok <= seg_tokens / HETIS_FINE_CHUNK_BELOW) ct = chunk_tokens / 2;
        if (n_tok <= seg_tokens / (4 * HETIS_FINE_CHUNK_BELOW)) ct = chunk_tokens / 4;
        ct = max(ct, 2 * kBlockTokens);
    }
    return ct;
}

// One step of the running combination of chunk results (o_c normalised, lse_c base 2) into
// (A, M, W): M' = max(M, lse_c), A' = A 2^(M-M') + o_c 2^(lse_c-M'), W' = W 2^(M-M') + 2^(lse_c-M').
// Written once, with explicit fused multiply-adds, because two code paths (the fold in LDS and
// the fold from the partial buffers) must produce the same bits.
struct FoldCoef {
    float Mn, so, sc;
};
__device__ __forceinline__ FoldCoef fold_coef(float Mo, float lc)
{
    FoldCoef f;
    f.Mn = fmaxf(Mo, lc);
    f.so = fast_exp2(Mo - f.Mn);
    f.sc = fast_exp2(lc - f.Mn);
    return f;
}
__device__ __forceinline__ float fold_weight(float Wo, const FoldCoef &f)
{
    return __builtin_fmaf(Wo, f.so, f.sc);
}
__device__ __forceinline__ float fold_elem(float y, float x, const FoldCoef &f)
{
    return __builtin_fmaf(y, f.so, x * f.sc);
}

// The R result rows of one chunk or segment in the registers of a wave: lane l holds elements
// 4 l + 256 k .. + 3 of the R * D, and with them the row's log-sum-exp.  With fewer than 256 elements
// the lanes beyond them hold copies of the last ones, which are not stored.
template <int D, int R>
struct RowRegs {
    static constexpr int K = (R * D + 255) / 256;
    f32x4 x[K];
    float lse[K];       // base 2
    __device__ static __forceinline__ int elem(int lane, int k) { return min(lane * 4 + k * 256, R * D - 4); }
    __device__ static __forceinline__ bool stored(int lane) { return R * D >= 256 || lane * 4 < R * D; }
    __device__ __forceinline__ void load(const float (*o)[D], const float *lse2, int lane)
    {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            x[k] = *reinterpret_cast<const f32x4 *>(&o[0][0] + elem(lane, k));
            lse[k] = lse2[elem(lane, k) / D];
        }
    }
};

// Result rows -> `out` (fp16) or the partial buffers (fp32, natural-log log-sum-exp).
template <int D, int R>
__device__ __forceinline__ void store_result(const RowRegs<D, R> &g, int kind, int64_t dest,
                                             const AttnParams &p, int lane)
{
    if (!RowRegs<D, R>::stored(lane)) return;
#pragma unroll
    for (int k = 0; k < RowRegs<D, R>::K; ++k) {
        const int idx = lane * 4 + k * 256, r = idx / D, d = idx % D;
        f32x4 v = g.x[k];
        if (kind == kKindPartial) {
            // the r rows of one (row, head, segment) are contiguous in the partial buffers
            *reinterpret_cast<f32x4 *>(p.o_partial + dest * (R * D) + idx) = v;
            if (d == 0) p.lse_partial[dest * R + r] = g.lse[k] * kLn2;
        } else {
            if (kind == kKindZero) v = f32x4{0.f, 0.f, 0.f, 0.f};
            union {
                __half2 h[2];
                uint2 u;
            } pk;
            pk.h[0] = __floats2half2_rn(v.x, v.y);
            pk.h[1] = __floats2half2_rn(v.z, v.w);
            *reinterpret_cast<uint2 *>(p.out + (dest + r) * D + d) = pk.u;
        }
    }
}

// Partial result of a segment that is merged inside this launch (AttnParams::arrivals): by
// whichever wave stores the row's last segment, possibly on another XCD, so the words are
// stored device-coherently, sixteen bytes a lane.
// `base2`: the log-sum-exp is stored as it is (chunk results of kModeSpread), otherwise as a
// natural logarithm (segment results).
template <int D, int R>
__device__ __forceinline__ void store_partial_coherent(const RowRegs<D, R> &g, int64_t dest,
                                                       const AttnParams &p, int lane, bool base2)
{
    const __amdgpu_buffer_rsrc_t dst = coherent_rsrc(p.o_partial + dest * (R * D), R * D * 4);
#pragma unroll
    for (int k = 0; k < RowRegs<D, R>::K; ++k) {
        const int idx = lane * 4 + k * 256;              // (past the R * D elements: not stored)
        coherent_store_b128(dst, idx * 4, __builtin_bit_cast(u32x4, g.x[k]));
        if (idx < R * D && idx % D == 0)
            coherent_store(p.lse_partial + dest * R + idx / D, base2 ? g.lse[k] : g.lse[k] * kLn2);
    }
}

// Partial results loaded together by the two functions below.  Their loads are device-coherent
// (the partial results may come from other XCDs) and the compiler keeps such loads in program
// order with every use, so a loop that loads and uses one result at a time pays a memory round
// trip for each: the wave that ends a launch then spends tens of microseconds on a row.
// With four or eight rows a result (kPartVectors) a lane loads vectors of four words, as many as there
// are registers for (sixteen with 8 x 128 words, four results; eight results go to scratch memory), and looks
// its row's weight up; four results together instead of two: 64 rows of 500 to 3000 tokens 19.4 -> 18.7 us, 8 of
// 500 to 1500 14.6 -> 14.0, the step of 144 pairs 41.6 -> 40.9, 300 rows of 100 to 600 21.2 -> 21.5;
// with one or two rows it loads words, the same dims of every row, and weights are the same in all lanes.
// A step of 144 pairs of 8-head groups: words 44.9 us, vectors 43.4; 16 chats x 13 heads (r = 1) 27.5 and 28.1.
// r = 4: vectors too, but half as many: more only fills registers, which are the streaming loop's as well
// (218 of them against 182 at 64 dims, 256 against 235 at 128).  Words / 16 vectors / 8, 64 dims: 160 rows
// of 500 to 2000 tokens 21.35 / 21.18 / 20.75 us, 508 of them 39.2 / 40.0 / 39.4; words / 16 / 8, 128 dims:
// 400 of 300 to 1200 40.5 / 40.3 / 39.7, 12 of 10k to 32k 32.6 / 32.5 / 32.8.
template <int R>
constexpr bool kPartVectors = R >= 4;
template <int D, int R>
constexpr int kPartBatch =                                         // at most 64 / R
    !kPartVectors<R> ? 16 : (R == 4 ? 8 : 16) / RowRegs<D, R>::K;

// Partial results in slots slot_of(0), slot_of(1), ... of the partial buffers -> x; their
// log-sum-exps come back with lane u * R + r holding that of result u, row r.
template <int D, int R, class SlotOf>
__device__ __forceinline__ float load_partials(const AttnParams &p, f32x4 (&x)[kPartBatch<D, R>][RowRegs<D, R>::K],
                                               SlotOf slot_of, int lane)
{
    const float lc = coherent_load(p.lse_partial + slot_of(min(lane / R, kPartBatch<D, R> - 1)) * R + lane % R);
    const int64_t s0 = slot_of(0);
    const __amdgpu_buffer_rsrc_t src = coherent_rsrc(
        p.o_partial + s0 * (R * D), uniform((int)(slot_of(kPartBatch<D, R> - 1) - s0 + 1) * (R * D * 4)));
#pragma unroll
    for (int u = 0; u < kPartBatch<D, R>; ++u) {
        const int from = uniform((int)(slot_of(u) - s0) * (R * D * 4));
#pragma unroll
        for (int k = 0; k < RowRegs<D, R>::K; ++k)
            x[u][k] = __builtin_bit_cast(
                f32x4, coherent_load_b128(src, RowRegs<D, R>::elem(lane, k) * 4, from));
    }
    return lc;
}

// x of lane `lane + ahead`
__device__ __forceinline__ float from_lane(float x, int lane, int ahead)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(4 * lane + 4 * ahead, __float_as_int(x)));
}

// Log-sum-exp merge of the n_segs partial results of one row, ascending segment order, by one
// wave: M = max_c lse_c, w_c = exp(lse_c - M), out = fp16(sum_c w_c o_c / sum_c w_c).  `first` is the
// index of segment 0 of the row in the partial buffers, segment c sits `stride` * c slots further.
// The maximum takes one load a lane per 64 log-sum-exps, the sums one round trip per
// kPartBatch segments (two rows of 5 to 7 segments per head, one load at a time: 25 us of the 70
// that launch took).
template <int D, int R>
__device__ __forceinline__ void merge_partials(const AttnParams &p, int64_t first, int n_segs,
                                               int stride, int64_t out_row, int lane)
{
    if constexpr (kPartVectors<R>) {
        first = uniform(first);
        n_segs = uniform(n_segs);
        constexpr int K = RowRegs<D, R>::K, U = kPartBatch<D, R>;
        const int64_t step = (int64_t)stride * R;        // rows of the buffers per segment
        const float *lse = p.lse_partial + first * R;    // [segment][r]
        // lane l looks at segments l / R, l / R + 64 / R, ... of row l % R
        float mx = -INFINITY;
#pragma unroll 1
        for (int c0 = 0; c0 < n_segs; c0 += 64 / R)
            mx = fmaxf(mx, coherent_load(lse + min(c0 + lane / R, n_segs - 1) * step + lane % R));
#pragma unroll
        for (int off = 32; off >= R; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        RowRegs<D, R> g;
        float M[K], W[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            M[k] = __shfl(mx, RowRegs<D, R>::elem(lane, k) / D, 64);
            W[k] = 0.f;
            g.x[k] = f32x4{0.f, 0.f, 0.f, 0.f};
            g.lse[k] = 0.f;
        }
#pragma unroll 1
        for (int c0 = 0; c0 < n_segs; c0 += U) {
            f32x4 x[U][K];
            const float lc = load_partials<D, R>(
                p, x, [&](int u) { return first + (int64_t)min(c0 + u, n_segs - 1) * stride; }, lane);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (c0 + u >= n_segs) continue;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const float lse_c = from_lane(lc, RowRegs<D, R>::elem(lane, k) / D, u * R);
                    const float w = fast_exp2((lse_c - M[k]) * kLog2e);
                    W[k] += w;
#pragma unroll
                    for (int e = 0; e < 4; ++e) g.x[k][e] = fmaf(w, x[u][k][e], g.x[k][e]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
#pragma unroll
            for (int e = 0; e < 4; ++e) g.x[k][e] /= W[k];
        }
        store_result<D, R>(g, kKindOut, out_row, p, lane);
    } else {
        constexpr int V = D / 64;                        // words per lane and row: 1 or 2
        constexpr int U = kPartBatch<D, R>;
        const int64_t step = (int64_t)stride * R;        // rows of the buffers per segment
        const float *lse = p.lse_partial + first * R;    // [segment][r]
        const float *op = p.o_partial + first * (R * D) + lane;
        // lane l looks at segments l / R, l / R + 64 / R, ... of row l % R
        float mx = -INFINITY;
#pragma unroll 1
        for (int c0 = 0; c0 < n_segs; c0 += 64 / R)
            mx = fmaxf(mx, coherent_load(lse + min(c0 + lane / R, n_segs - 1) * step + lane % R));
#pragma unroll
        for (int off = 32; off >= R; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        float M[R], W[R], acc[R][V];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            M[r] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mx), r));
            W[r] = 0.f;
#pragma unroll
            for (int v = 0; v < V; ++v) acc[r][v] = 0.f;
        }
#pragma unroll 1
        for (int c0 = 0; c0 < n_segs; c0 += U) {
            float x[U][R][V];
            // lane u * R + r: log-sum-exp of segment c0 + u, row r
            const int lc = __float_as_int(coherent_load(lse + min(c0 + lane / R, n_segs - 1) * step + lane % R));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t row = min(c0 + u, n_segs - 1) * step;
#pragma unroll
                for (int r = 0; r < R; ++r) {
#pragma unroll
                    for (int v = 0; v < V; ++v) x[u][r][v] = coherent_load(op + (row + r) * D + v * 64);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (c0 + u >= n_segs) continue;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float lse_c = __int_as_float(__builtin_amdgcn_readlane(lc, u * R + r));
                    const float w = fast_exp2((lse_c - M[r]) * kLog2e);
                    W[r] += w;
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[r][v] = fmaf(w, x[u][r][v], acc[r][v]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            __half *dst = p.out + (out_row + r) * D + lane;
#pragma unroll
            for (int v = 0; v < V; ++v) dst[v * 64] = __float2half_rn(acc[r][v] / W[r]);
        }
    }
}

// kModeSpread: the ns chunk results of one segment lie in the partial buffers (chunk c in slot
// slot0 + c, log-sum-exp base 2).  One wave combines them with the operations a workgroup
// applies to the chunks of a segment in kModeSegments, in the same order: folded in ascending
// order, then normalised.  `whole_row`: the segment is the whole row and the result goes to
// `out`; otherwise it replaces the first chunk result in the buffers, as the partial result of
// the segment (natural-log log-sum-exp) that merge_partials expects.
template <int D, int R>
__device__ __forceinline__ void fold_segment_from_chunks(const AttnParams &p, int64_t slot0, int ns,
                                                         bool whole_row, int64_t out_row, int lane)
{
    if constexpr (kPartVectors<R>) {
        slot0 = uniform(slot0);
        ns = uniform(ns);
        constexpr int K = RowRegs<D, R>::K, U = kPartBatch<D, R>;
        RowRegs<D, R> g;
        float W[K];
#pragma unroll 1
        for (int c0 = 0; c0 < ns; c0 += U) {
            f32x4 x[U][K];
            const float lc = load_partials<D, R>(p, x, [&](int u) { return slot0 + min(c0 + u, ns - 1); }, lane);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (c0 + u >= ns) continue;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const float lse_c = from_lane(lc, RowRegs<D, R>::elem(lane, k) / D, u * R);
                    if (c0 + u == 0) {
                        g.lse[k] = lse_c;
                        W[k] = 1.f;
                        g.x[k] = x[u][k];
                    } else {
                        const FoldCoef f = fold_coef(g.lse[k], lse_c);
                        W[k] = fold_weight(W[k], f);
                        g.lse[k] = f.Mn;
#pragma unroll
                        for (int e = 0; e < 4; ++e) g.x[k][e] = fold_elem(g.x[k][e], x[u][k][e], f);
                    }
                }
            }
        }
        if (ns > 1) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float inv = __builtin_amdgcn_rcpf(W[k]);
                g.lse[k] = g.lse[k] + fast_log2(W[k]);
#pragma unroll
                for (int e = 0; e < 4; ++e) g.x[k][e] *= inv;
            }
        }
        if (whole_row)
            store_result<D, R>(g, kKindOut, out_row, p, lane);
        else
            store_partial_coherent<D, R>(g, slot0, p, lane, false);
    } else {
        constexpr int V = D / 64;
        constexpr int U = kPartBatch<D, R>;
        float a[R][V], M[R], W[R];
#pragma unroll 1
        for (int c0 = 0; c0 < ns; c0 += U) {
            float x[U][R][V];
            // lane u * R + r: log-sum-exp of chunk c0 + u, row r
            const int lc = __float_as_int(
                coherent_load(p.lse_partial + (slot0 + min(c0 + lane / R, ns - 1)) * R + lane % R));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t slot = slot0 + min(c0 + u, ns - 1);
#pragma unroll
                for (int r = 0; r < R; ++r) {
#pragma unroll
                    for (int v = 0; v < V; ++v)
                        x[u][r][v] = coherent_load(p.o_partial + (slot * R + r) * D + v * 64 + lane);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (c0 + u >= ns) continue;
                    const float lse_c = __int_as_float(__builtin_amdgcn_readlane(lc, u * R + r));
                    if (c0 + u == 0) {
                        M[r] = lse_c;
                        W[r] = 1.f;
#pragma unroll
                        for (int v = 0; v < V; ++v) a[r][v] = x[u][r][v];
                    } else {
                        const FoldCoef f = fold_coef(M[r], lse_c);
                        W[r] = fold_weight(W[r], f);
                        M[r] = f.Mn;
#pragma unroll
                        for (int v = 0; v < V; ++v) a[r][v] = fold_elem(a[r][v], x[u][r][v], f);
                    }
                }
            }
        }
        if (ns > 1) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float s = __builtin_amdgcn_rcpf(W[r]);
                M[r] = M[r] + fast_log2(W[r]);
#pragma unroll
                for (int v = 0; v < V; ++v) a[r][v] *= s;
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (whole_row) {
                __half *dst = p.out + (out_row + r) * D + lane;
#pragma unroll
                for (int v = 0; v < V; ++v) dst[v * 64] = __float2half_rn(a[r][v]);
            } else {
#pragma unroll
                for (int v = 0; v < V; ++v)
                    coherent_store(p.o_partial + (slot0 * R + r) * D + v * 64 + lane, a[r][v]);
                if (lane == 0) coherent_store(p.lse_partial + slot0 * R + r, M[r] * kLn2);
            }
        }
    }
}

__host__ __device__ constexpr size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

__device__ __forceinline__ int mail_load(const int *flag)
{
    return __hip_atomic_load(flag, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void mail_store(int *flag, int v)
{
    __hip_atomic_store(flag, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// Orders the LDS accesses of one wave around a point where lanes read what other lanes of
// the same wave wrote (the hardware keeps a wave's LDS operations in order; this keeps the
// compiler from moving them).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The new token's K row and V row of (sequence, KV head g) -> slot pos % 16 of the tile
// (block, g); lanes [0, D/8) move the K row, the next D/8 lanes the V row, 16 bytes each; nothing
// is read or written unless `inside`.
template <int D>
__device__ __forceinline__ void store_new_rows(const AttnParams &p, int seq, int g, int64_t tile_off,
                                               int slot, int n_kv_heads, int lane, bool inside)
{
    constexpr int LR = D / 8;
    if (lane < 2 * LR && inside) {
        const bool is_v = lane >= LR;
        const int c = lane % LR;
        const __half *src = (is_v ? p.v_new : p.k_new) + ((int64_t)seq * n_kv_heads + g) * D + c * 8;
        __half *dst = const_cast<__half *>(is_v ? p.v_cache : p.k_cache) + tile_off + slot * D + c * 8;
        *reinterpret_cast<uint4 *>(dst) = *reinterpret_cast<const uint4 *>(src);
    }
}

// Launch of fewer than kMaxQuickRows rows of one segment each, the longest of more than one full
// chunk: are its chunks handed out singly (true), or the rows whole, one or two a workgroup?
// `rows` rows of `tokens` tokens in all and `longest` at most, `chunks` chunks; G workgroups.
// Whole rows wait for the longest one, or, with more rows than workgroups, for two in turn, beside
// idle compute units; but their chunks meet in LDS, where the results of single ones go through
// global memory, r times as much with r query rows.  Measured with either side forced, rows whole ->
// single chunks, in us (r = 1, 128 dims, lengths uniform, unless stated):
//  - Up to G rows.  What idles is 1 - tokens / (G * longest).  r < 4: chunks, unless less than
//    three tenths idle and some wave would take a second chunk (128 rows of 4096: 52.6 -> 50.6; 255 of
//    275 to 1100 23.3 -> 22.8; but 230 of 600 17.8 -> 20.4, 255 of 4096 92.7 -> 95.2).  r >= 4: a row
//    of up to NW chunks is one turn of a workgroup; it gains when it is several chunks long, the
//    more the more idles (r = 8, 200 rows of 500 to 2000: 41.3 -> 36.0; 300 to 1200: 25.8 -> 28.9;
//    250 to 1000, whose chunks are half as long: 25.0 -> 23.5; 150 to 600: 17.8 -> 17.7).
//  - More rows.  Chunks for a few long ones among short ones (511 rows, log-normal around 820, up
//    to 4096: 67.5 -> 57.6), where the rows are alike and the workgroups' second turn is mostly empty
//    (270 of 4096: 120 -> 99), and for up to one (r >= 4) or some 2.4 chunks a wave (390 of 1200: 49.0 ->
//    45.3; 480 of 75 to 300, r = 2: 19.8 -> 19.5, 480 of up to 290: 23.0 -> 17.6; but around 2.5 a wave 460
//    of 275 to 1100 34.7 -> 37.6, 64 dims 23.8 -> 29.0).  Otherwise rows whole: 511 of 500 to 2000 57.6 ->
//    61.9, r = 2 59.2 -> 65.6, r = 8 61.4 -> 68.8; of 150 to 600, r = 8, 26.2 -> 32.4.
//  - r >= 4 and rows of more than one turn, G or more of them: whole, as when that was the faster way
//    everywhere.  It no longer is (r = 8, 360 of 750 to 3000: 70.0 -> 70.5, but 270 of 4096 143 -> 114,
//    256 log-normal around 820 68 -> 40, 511 of these 78.8 -> 64.5).
template <int D, int R, int NW>
__device__ __forceinline__ bool spread_pays(int G, int rows, int longest, int tokens, int chunks)
{
    constexpr int ct = decode_chunk_tokens(R), turn = NW * ct;      // tokens a workgroup's waves hold
    const int waves = NW * G, full = G * longest;
    const bool idle = 10 * tokens < 7 * full;
    if (rows <= G) {
        if (R < 4) return idle || chunks <= waves;
        if (!idle || (rows == G && longest > turn)) return false;
        // chunks of the longest row are full ones, or half as long
        const bool halves = chunk_tokens_of(longest, ct, decode_seg_tokens(R)) < ct;
        return (!halves && 10 * chunks <= 4 * waves) ||
               200ll * ct * tokens < (halves ? 60ll : 35ll) * longest * full;
    }
    constexpr bool wide = R < 4 && R * D > 128;             // a partial result of more than 512 bytes
    const bool even = 20 * tokens >= 17 * full && 16 * rows < (wide ? 24 : 26) * G;
    if (R < 4) return idle || even || 10 * chunks <= (wide ? 23 : 25) * waves;
    return longest <= turn && (chunks <= waves || 20 * tokens < (R * D <= 512 ? 18 : 11) * full || even);
}

// Counters (AttnParams::arrivals), n_rows = (enumeration rows) x (selected heads) of the launch:
// entry row counts the stored segment results of that row; in kModeSpread entry
// n_rows + row * (segments per row the buffers provide for) + j counts the stored chunk results
// of segment j of that row.  There the wave that completes a segment folds its chunks, which
// spreads the folding of a long row over as many waves as it has segments, stores the segment
// result and counts it in for the row in turn.
template <int R>
__device__ __forceinline__ int64_t arrival_counter(const AttnParams &p, int dest, bool spread, int n_rows)
{
    constexpr int gc = decode_seg_tokens(R) / decode_chunk_tokens(R);
    const int row = dest / p.max_segs;               // (enumeration row, head)
    return spread ? n_rows + (int64_t)row * (p.max_segs / gc) + (dest - row * p.max_segs) / gc : row;
}

// What follows a count: `before` is the counter's value before `added` results were counted in.  All
// arguments are the same in every lane.
template <int D, int R>
__device__ __forceinline__ void combine_if_last(const AttnParams &p, int before, int added, int dest, int parts,
                                                int64_t out_row, int len, bool spread, int n_rows,
                                                int lane)
{
    // what follows from the lane's number is worked out here: hoisted out of the writer wave's loop, it
    // takes more registers than there are
    asm volatile("" : "+v"(lane));
    constexpr int seg_tokens = decode_seg_tokens(R), gc = seg_tokens / decode_chunk_tokens(R);
    const int64_t row = dest / p.max_segs;
    int n_segs = parts;
    if (spread) {
        const int j = (dest - (int)row * p.max_segs) / gc;
        const int n_tok = min(seg_tokens, len - j * seg_tokens);
        const int ct = chunk_tokens_of(n_tok, decode_chunk_tokens(R), seg_tokens);
        const int ns = udiv(n_tok + ct - 1, ct);
        if (before + added != ns) return;
        n_segs = (len + seg_tokens - 1) / seg_tokens;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        fold_segment_from_chunks<D, R>(p, row * p.max_segs + j * gc, ns,
                                       n_segs == 1, out_row, lane);
        unsigned seen = 0;
        if (n_segs > 1) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);           // the segment result is stored
        }
        if (lane == 0) {
            __hip_atomic_store(p.arrivals + arrival_counter<R>(p, dest, true, n_rows), 0u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            if (n_segs > 1)
                seen = __hip_atomic_fetch_add(p.arrivals + row, 1u, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
        }
        if (n_segs == 1 || (int)__builtin_amdgcn_readfirstlane(seen) + 1 != n_segs) return;
    } else if (before + added != n_segs) {
        return;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    merge_partials<D, R>(p, row * p.max_segs, n_segs, spread ? gc : 1, out_row, lane);
    if (lane == 0)
        __hip_atomic_store(p.arrivals + row, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace hetis
