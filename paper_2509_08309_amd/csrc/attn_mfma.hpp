// MFMA arithmetic for grouped-query attention (r query heads share one KV head): here a
// tile is a real dense contraction, [16 tokens x D] against [D x r] and [D x 16 tokens]
// against [16 tokens x r], so it goes to the matrix cores with the query group padded to 16
// columns.  Both products are taken transposed so that the softmax output of the first is,
// lane for lane, the B operand of the second:
//
//   S^T = K . Q^T      v_mfma_f32_16x16x32_f16, D/32 steps
//         A = K tile : lane l holds K[token l%16][dims (l/16)*8 + 32*step .. +8]  (a 16-byte
//                      load straight from the cache tile; staging K through LDS with
//                      row-coalesced loads was measured and made no difference)
//         B = Q^T    : lane l holds Q[head l%16][same dims]; heads >= r are zero columns
//         C          : lane l, reg i = score of token (l/16)*4 + i for head l%16
//   O^T += V^T . P     v_mfma_f32_16x16x16_f16, D/16 row blocks
//         B = P      : lane l holds p[token (l/16)*4 + i][head l%16], i = 0..3: exactly the
//                      C registers above after exp2 and conversion to fp16
//         A = V^T    : lane l holds V[token (l/16)*4 + i][dim of row l%16], i = 0..3: four tokens of
//                      one dim.  Lane l loads, of each of its four tokens, the D/16 dims from
//                      (l%16) * D/16 on (16 lanes a token row) and puts the halves of four tokens
//                      together in its own registers (v_perm_b32): row l%16 of block e is dim
//                      (l%16) * D/16 + e, so no lane needs a value that another one has loaded.
//         C          : lane l, reg i of block e = O[head l%16][dim ((l/16)*4 + i) * D/16 + e]
//
// Online softmax state per head lives in the 4 lanes {l%16 == head}: the running maximum is
// kept identical in all four (two cross-lane maxima per tile), the running sum is kept per
// lane group and added up once per chunk.
#pragma once
#include "attn_common.hpp"
#include "attn_persist.hpp"

namespace hetis {

typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef short i16x4 __attribute__((ext_vector_type(4)));

template <int D_, int R_>
struct MfmaPolicy {
    static constexpr int D = D_;
    static constexpr int R = R_;
    static_assert(D % 32 == 0 && R <= 16, "MFMA tiling");
    static constexpr int KS = D / 32;                 // contraction steps of S^T = K.Q^T
    static constexpr int MB = D / 16;                 // 16-dim row blocks of O^T
    static constexpr int WV = D / 32;                 // words of V a lane holds of each of its tokens
    // Wave-private LDS: the query rows of the current item.
    static constexpr int kQBytes = R * D * 2;
    static constexpr int kWaveLdsBytes = kQBytes;
    static constexpr int kWavesPerEu = 2;             // register budget: 512 / 2 per lane
    // Tile pairs in flight per wave: 16 KB at 64 dims, 24 KB at 128 (a piece of eight tiles then ends inside a turn).
    // 16 KB -> 24 KB at 128 dims: 160 rows of 300 to 1200 tokens, r = 8, 25.6 -> 24.0 us, r = 4 24.7 -> 23.0, 26 of
    // 150 to 18 700, r = 4, 26.5 -> 24.4, 768 of 2176, r = 8, 139.7 -> 138.6; but 12 of 10k to 32k, r = 8, 32.5 -> 32.9,
    // 300 of 100 to 600 20.9 -> 21.3.  (32 KB, while a chunk was one piece: slower throughout.)
    static constexpr int ring(bool) { return D_ == 64 ? 4 : 3; }
    // In split calls, whose chunks are one piece, short loops count for more: 24 rows of up to 26 tokens of 64 dims
    // (r = 4) 10.6 us with four pairs, 9.9 with three, 9.7 with two; 240 of up to 200 15.1, 14.2, 14.1; 24 of 300 to
    // 900 21.1, 20.6, 20.4; but 160 of 4k to 16k 81.0, 80.7, 83.3.  128 dims, three and two: 24 of up to 26 10.9 and
    // 10.5, of 300 to 900 34.1 and 33.6; 160 of 4k to 16k 141.2 and 143.9 (r = 8 149.8 and 150.3).
    static constexpr int ring_split = D_ == 64 ? 3 : 2;

    // of a team's wave: two copies of the arithmetic of a tile (4: 16 rows of 300 to 1200, r = 4, 16.8 -> 17.7)
    static constexpr int kTeamRing = 2;
    typedef unsigned int VWords __attribute__((ext_vector_type(WV)));
    struct Tile {
        u32x4 k[KS];
        VWords v[4];      // of token (l/16)*4 + i
    };
    struct Query {
        f16x8 b[KS];
    };
    struct State {
        float m;          // running maximum (base-2 domain) of head l%16
        float l;          // running sum over the tokens this lane group has seen
        f32x4 acc[MB];
    };

    __device__ static __forceinline__ void issue(Tile &t, __amdgpu_buffer_rsrc_t rk,
                                                 __amdgpu_buffer_rsrc_t rv, int lane)
    {
        const int koff = (lane & 15) * (2 * D) + (lane >> 4) * 16;
#pragma unroll
        for (int s = 0; s < KS; ++s) t.k[s] = buffer_load_u4(rk, koff + s * 64);
        const int voff = (lane >> 4) * (8 * D) + (lane & 15) * (4 * WV);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (WV == 4)
                t.v[i] = buffer_load_u4(rv, voff + i * (2 * D));
            else
                t.v[i] = buffer_load_u2(rv, voff + i * (2 * D));
        }
    }

    // Query rows: fetched as raw bytes one item ahead (kQBytes over 64 lanes), then passed
    // through the wave's LDS area into operand layout with zero columns for heads >= r.
    // (two named members instead of an array: the array form was kept in scratch memory when it
    // had two elements, and a scratch store in a streaming wave is a global store like any other)
    static constexpr int kQVec = (kQBytes / 16 + 63) / 64;
    static_assert(kQVec <= 2, "query rows of one group: at most 2 x 64 x 16 bytes");
    struct QueryPrefetch {
        u32x4 raw0, raw1;
    };
    __device__ static __forceinline__ void q_prefetch(QueryPrefetch &pre, const __half *rows, int lane)
    {
        const u32x4 *src = reinterpret_cast<const u32x4 *>(rows);
        pre.raw0 = src[min(lane, kQBytes / 16 - 1)];
        pre.raw1 = kQVec > 1 ? src[min(lane + 64, kQBytes / 16 - 1)] : u32x4{0u, 0u, 0u, 0u};
    }
    __device__ static __forceinline__ void q_commit(Query &q, const QueryPrefetch &pre,
                                                    unsigned char *stage, int lane)
    {
        u32x4 *dst = reinterpret_cast<u32x4 *>(stage);
        if (lane < kQBytes / 16) dst[lane] = pre.raw0;
        if (kQVec > 1 && lane + 64 < kQBytes / 16) dst[lane + 64] = pre.raw1;
        const int j = lane & 15;
        const __half *src =
            reinterpret_cast<const __half *>(stage) + min(j, R - 1) * D + (lane >> 4) * 8;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            u32x4 t = *reinterpret_cast<const u32x4 *>(src + s * 32);
            if (j >= R) t = u32x4{0u, 0u, 0u, 0u};
            q.b[s] = __builtin_bit_cast(f16x8, t);
        }
    }

    __device__ static __forceinline__ void reset(State &st)
    {
        st.m = kNegBig;
        st.l = 0.f;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) st.acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // What bounds a wave is the chain of dependent instructions of a tile, not the matrix cores, so the
    // chain is kept short: the scores in two chains of products, the maximum over the lane groups by the
    // swaps of the vector ALU instead of two trips through LDS, V^T put together in registers instead of
    // written to LDS and read back (the compiler waited for each of the eight reads in turn), the sums
    // brought to a new maximum only in tiles that have one.  One request of 1000 tokens, 2 groups of 8
    // heads of 128 dims x 4 20.7 -> 18.1 us, 16 x 4 groups of 4 heads of 128 20.5 -> 18.0, of 64 16.6 ->
    // 15.2, 16 x 4 of 8 heads, 700 to 2000 tokens, 22.1 -> 20.3; 768 rows of 2176, which wait for HBM,
    // within 1 %, but 800 rows of 1100 of 64 dims (r = 4; eight bytes a load) 46.0 -> 46.5.  Letting the
    // maximum lag behind by up to 8 saves another 3 % of the small ones, but the largest weight is then no
    // longer exactly 1 in fp16: error against 64 bits 2.9e-4 instead of 2.7e-4.
    template <int MAYBE_RAGGED>
    __device__ static __forceinline__ void update(State &st, const Tile &t, const Query &q,
                                                  float scale_log2, int lane, int n_valid)
    {
#pragma clang fp contract(off)
        // (two copies of this code must produce the same bits)
        const int grp = lane >> 4;
        // ---- scores of 16 tokens x 16 (padded) heads, in two chains of products
        f32x4 c = {0.f, 0.f, 0.f, 0.f}, c2 = c;
#pragma unroll
        for (int s = 0; s < KS; s += 2) {
            c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, t.k[s]), q.b[s], c, 0, 0, 0);
            c2 = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, t.k[s + 1]), q.b[s + 1], c2, 0, 0, 0);
        }
        c += c2;
        float s4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool valid = !MAYBE_RAGGED || grp * 4 + i < n_valid;
            s4[i] = valid ? c[i] * scale_log2 : -INFINITY;
        }
        float mt = fmaxf(fmaxf(s4[0], s4[1]), fmaxf(s4[2], s4[3]));
        mt = max_xor32(max_xor16(mt));
        if (__builtin_amdgcn_ballot_w64(mt > st.m) != 0) {
            const float m_new = fmaxf(st.m, mt);
            const float alpha = fast_exp2(st.m - m_new);
            st.m = m_new;
            st.l *= alpha;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) st.acc[mb] *= alpha;
        }
        float p4[4];
        float ps = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p4[i] = fast_exp2(s4[i] - st.m);
            ps += p4[i];
        }
        st.l += ps;
        const f16x4 pb = {(_Float16)p4[0], (_Float16)p4[1], (_Float16)p4[2], (_Float16)p4[3]};
        // ---- O^T += V^T . P
        // (rows past n_valid were loaded as zeros: see tile_rsrc)
        const VWords *v = t.v;
#pragma unroll
        for (int e = 0; e < MB; ++e) {
            const unsigned sel = e % 2 ? 0x07060302u : 0x05040100u;
            const u32x2 vt = {__builtin_amdgcn_perm(v[1][e / 2], v[0][e / 2], sel),
                              __builtin_amdgcn_perm(v[3][e / 2], v[2][e / 2], sel)};
            st.acc[e] = __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, vt), pb, st.acc[e], 0, 0, 0);
        }
    }

    // state of one piece into the state of the pieces before it, lane by lane (sums that are scaled in place:
    // with the products the other way round every register took a move as well)
    __device__ static __forceinline__ void fold(State &tot, const State &st)
    {
#pragma clang fp contract(off)
        const float M = fmaxf(tot.m, st.m);
        const float a = fast_exp2(tot.m - M), b = fast_exp2(st.m - M);
        tot.m = M;
        tot.l = __builtin_fmaf(st.l, b, tot.l * a);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int e = 0; e < 4; ++e) tot.acc[mb][e] = __builtin_fmaf(st.acc[mb][e], b, tot.acc[mb][e] * a);
    }
    __device__ static __forceinline__ void settle(State &) {}           // (no piece is one turn)
    // state <-> LDS, sixteen bytes a lane at a time
    static constexpr int kStateVecs = MB + 1;
    __device__ static __forceinline__ void deposit(const State &st, f32x4 *to, int lane)
    {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) to[mb * 64 + lane] = st.acc[mb];
        to[MB * 64 + lane] = f32x4{st.m, st.l, 0.f, 0.f};
    }
    __device__ static __forceinline__ void collect(State &st, const f32x4 *from, int lane)
    {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) st.acc[mb] = from[mb * 64 + lane];
        const f32x4 ml = from[MB * 64 + lane];
        st.m = ml.x;
        st.l = ml.y;
    }
    // normalised rows and their base-2 log-sum-exp -> LDS (the wave's mailbox)
    __device__ static __forceinline__ void finish(State &st, float (&o)[R][D], float (&lse)[R],
                                                  int lane)
    {
        const int j = lane & 15, grp = lane >> 4;
        float l = st.l;
        l = sum_xor32(sum_xor16(l));
        if (j < R) {
            const float inv = __builtin_amdgcn_rcpf(l);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < MB; e += 4) {
                    const float4 v = make_float4(st.acc[e][i] * inv, st.acc[e + 1][i] * inv,
                                                 st.acc[e + 2][i] * inv, st.acc[e + 3][i] * inv);
                    *reinterpret_cast<float4 *>(&o[j][(grp * 4 + i) * MB + e]) = v;
                }
            if (grp == 0) lse[j] = st.m + fast_log2(l);
        }
    }
};

}  // namespace hetis
