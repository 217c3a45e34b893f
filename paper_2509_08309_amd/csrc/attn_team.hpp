// Launches of few rows: the waves of a workgroup as a team on one piece of work.
//
// Where there is at most one full chunk of work for a workgroup, a launch is bound by the chain of what one
// wave does: the tiles of its chunk one after the other, then the round trips of the combination.  So the unit
// handed out is the ITEM, a window of one full chunk (chunk_tokens) of a row, and the NW streaming waves
// of a workgroup compute its NW pieces (decode_piece_tokens) side by side.  A wave leaves the state of its
// piece in LDS (deposit); the fifth wave, the MERGER, folds the states of a chunk's pieces in ascending order,
// with the operations a single wave applies to them in the other launches, and takes the result further:
//  - rows of which one workgroup has everything: folded on in registers, as the writer wave of the
//    other launches does in LDS, and stored as the fp16 row;
//  - other rows: chunk results go to the partial buffers (device-coherent stores) and are counted in; the
//    merger whose count completes a segment folds its chunks, and whoever completes a row merges the
//    segments (combine_if_last).
// Rows of up to a window that are cut into chunks of one piece: the wave finishes its chunk itself and leaves
// the rows in LDS, so that the merger has one fold a chunk to do instead of the whole of it four times over (16 rows
// of 17 to 255 tokens of 64 dims 7.2 -> 5.5 us, 256 of 100 to 256 9.3 -> 8.0, 16 of 17 to 255, r = 8, 8.8 -> 7.9).
// Nothing in a result shows who computed what: the cut into chunks and pieces is a function of the
// row's length, and every fold has a fixed order.
//
// A workgroup has one item, or (`whole`) all items of one row, one after the other; nothing is drawn, and
// nobody is waited for outside the workgroup.  A state's slot in LDS is EMPTY -> the wave fills it -> FULL ->
// the merger reads it -> EMPTY; states are deposited and folded in the same order, so the earliest one not
// yet folded can always be deposited.  Every wait is bounded all the same (see kSpinLimit).
// Decode step with the store folded in: the wave whose piece holds position L - 1 stores the new token's
// rows before its first load.
#pragma once
#include "attn_combine.hpp"

namespace hetis {

struct TeamItem {
    int b, g, seq;      // enumeration row (sequence, or pair), KV head, sequence of q / out rows
    int row;            // (enumeration row, selected head): index of the row in the partial buffers
    int t0, len;        // first token of the window; tokens of the row
};

template <class Policy, int NW>
struct alignas(16) TeamLds {
    f32x4 state[2][NW][Policy::kStateVecs * 64];        // a wave may be two items ahead of the merger
    unsigned char staging[NW][Policy::kWaveLdsBytes ? Policy::kWaveLdsBytes : 16];
    float o[Policy::R][Policy::D];      // rows of a chunk on their way into the merger's registers
    float lse[Policy::R];
    // a chunk of one piece: its wave leaves the finished rows, not the state
    struct Rows {
        float o[Policy::R][Policy::D], lse[Policy::R];
    } rows[NW];
};

// The fold of a row's chunk results, in ascending order, in the registers of one wave.
template <int D, int R>
struct RowFold {
    static constexpr int K = RowRegs<D, R>::K;
    RowRegs<D, R> y;
    float W[K];
    __device__ __forceinline__ void take_in(const RowRegs<D, R> &g, int c)      // chunk c of the row
    {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (c == 0) {
                y.x[k] = g.x[k];
                y.lse[k] = g.lse[k];
                W[k] = 1.f;
            } else {
                const FoldCoef f = fold_coef(y.lse[k], g.lse[k]);
                y.lse[k] = f.Mn;
                W[k] = fold_weight(W[k], f);
                y.x[k] = f32x4{fold_elem(y.x[k].x, g.x[k].x, f), fold_elem(y.x[k].y, g.x[k].y, f),
                               fold_elem(y.x[k].z, g.x[k].z, f), fold_elem(y.x[k].w, g.x[k].w, f)};
            }
        }
    }
    __device__ __forceinline__ void store(int64_t out_row, int n_chunks, const AttnParams &p, int lane)
    {
        if (n_chunks > 1) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float inv = __builtin_amdgcn_rcpf(W[k]);
                y.x[k] = f32x4{y.x[k].x * inv, y.x[k].y * inv, y.x[k].z * inv, y.x[k].w * inv};
            }
        }
        store_result<D, R>(y, kKindOut, out_row, p, lane);
    }
};

// A wave's pieces of a row, in ascending order: piece t, of t < T, is the tokens from first.t0 + t * step, as
// many as a piece has.  on_piece(state, t) takes the state of each that holds a token.  Decode step with the
// store folded in: the wave whose piece holds position L - 1 stores the new token's rows before its first load.
template <class Policy, bool PAIRS, class OnPiece>
__device__ __forceinline__ void run_pieces(const AttnParams &p, const TeamItem &first, int T, int step,
                                           unsigned char *staging, int lane, const OnPiece &on_piece)
{
    constexpr int D = Policy::D, R = Policy::R;
    constexpr int kPiece = decode_piece_tokens(R);
    const int len = first.len;
    constexpr int RING = Policy::kTeamRing, PT = kPiece / kBlockTokens;
    static_assert(PT % RING == 0, "a piece is whole turns of the ring");
    const int64_t head_off = PAIRS ? 0 : (int64_t)first.g * p.stride_head;          // pairs: single-head tiles
    // Block ids by scalar loads, which are counted apart from the tiles: a vector load would come back
    // behind the tiles already asked for, and the refill that needs it would find nothing in flight.
    const auto *bt = (const __attribute__((address_space(4))) int32_t *)(uintptr_t)(
        p.block_table + (int64_t)first.b * p.max_blocks_per_seq);
    auto piece_tokens = [&](int t) { return t < T ? min(kPiece, max(0, len - first.t0 - t * step)) : 0; };
    auto fill = [&](int t, int n_tok, int (&ids)[PT]) {
        const int j0 = n_tok > 0 ? (first.t0 + t * step) / kBlockTokens : 0;
        const int last = max((n_tok + kBlockTokens - 1) / kBlockTokens - 1, 0);
#pragma unroll
        for (int i = 0; i < PT; ++i) ids[i] = bt[min(j0 + min(i, last), p.max_blocks_per_seq - 1)];
    };
    auto issue = [&](typename Policy::Tile &t, int blk, int idx, int n_tok) {
        const int64_t base = (int64_t)blk * p.stride_block + head_off;
        const int nbytes = min(kBlockTokens, max(0, n_tok - idx * kBlockTokens)) * (2 * D);
        Policy::issue(t, tile_rsrc(p.k_cache + base, nbytes), tile_rsrc(p.v_cache + base, nbytes), lane);
    };
    int n_tok = piece_tokens(0), ids[PT], next_ids[PT];
    fill(0, n_tok, ids);
    if (p.k_new != nullptr && len > 0) {
        // the new token's rows.  Like a store on its own it leaves out a row whose position is past its
        // block table, whose head does not exist or whose block id is negative.
        const int pos = len - 1, behind = pos - first.t0;
        const int t_new = udiv(max(behind, 0), step);
        if (behind >= 0 && t_new < T && behind - t_new * step < kPiece) {
            const int jb = pos / kBlockTokens, n_kv_heads = p.n_q_heads / R;
            const int blk = bt[min(jb, p.max_blocks_per_seq - 1)];
            const bool inside = (jb < p.max_blocks_per_seq) & ((unsigned)first.g < (unsigned)n_kv_heads) & (blk >= 0);
            store_new_rows<D>(p, first.seq, first.g, (int64_t)blk * p.stride_block + head_off, pos % kBlockTokens,
                              n_kv_heads, lane, inside);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);
        }
    }
    typename Policy::Query q;
    typename Policy::QueryPrefetch q_pre;
    typename Policy::Tile ring[RING];
    Policy::q_prefetch(q_pre, p.q + ((int64_t)first.seq * p.n_q_heads + first.g * R) * D, lane);
#pragma unroll
    for (int s = 0; s < RING; ++s) issue(ring[s], ids[s], s, n_tok);
    Policy::q_commit(q, q_pre, staging, lane);
    typename Policy::State st;
#pragma unroll 1
    for (int t = 0; t < T; ++t) {
        const int n_next = piece_tokens(t + 1);
        fill(t + 1, n_next, next_ids);
        Policy::reset(st);
        const int n_my = (n_tok + kBlockTokens - 1) / kBlockTokens;
        const int lim = max(RING, (n_my + RING - 1) / RING * RING);      // tiles, as whole ring turns
        // Two copies of the tile's arithmetic per slot: code that runs a few times costs what it takes to
        // fetch it.  (Scheduling fences as in the other launches: consume a slot, refill it at once.)
        int i = 0;
#pragma unroll 1
        for (; PT > RING && i + RING < lim; i += RING) {
#pragma unroll
            for (int s = 0; s < RING; ++s) {
                Policy::template update<kOneCopy>(st, ring[s], q, p.scale_log2, lane, n_tok - (i + s) * kBlockTokens);
                __builtin_amdgcn_sched_barrier(0);
                issue(ring[s], ids[RING + s], i + RING + s, n_tok);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int k = 0; k + RING < PT; ++k) ids[k] = ids[k + RING];  // tile i + RING comes first
        }
#pragma unroll
        for (int s = 0; s < RING; ++s) {
            if (i + s < n_my)
                Policy::template update<kOneCopy>(st, ring[s], q, p.scale_log2, lane, n_tok - (i + s) * kBlockTokens);
            __builtin_amdgcn_sched_barrier(0);
            issue(ring[s], next_ids[s], s, n_next);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (n_tok > 0) on_piece(st, t);
        n_tok = n_next;
#pragma unroll
        for (int k = 0; k < PT; ++k) ids[k] = next_ids[k];
    }
}

// The workgroup's part of such a launch.  `full`: 2 NW words in LDS, kMailEmpty, and everybody knows it;
// n_rows: (enumeration rows) x (selected heads) of the launch; `spread`: what the launch goes by in
// AttnParams::control.
template <class Policy, int NW, bool PAIRS>
__device__ __forceinline__ void team_run(const AttnParams &p, const TeamItem &first, bool whole, bool spread,
                                         int n_rows, int *full, unsigned char *smem)
{
    constexpr int D = Policy::D, R = Policy::R;
    constexpr int kWindow = decode_chunk_tokens(R), kPiece = decode_piece_tokens(R);
    constexpr int kSeg = decode_seg_tokens(R), gc = kSeg / kWindow;
    static_assert(NW * kPiece == kWindow, "a piece a wave");
    TeamLds<Policy, NW> &l = *reinterpret_cast<TeamLds<Policy, NW> *>(smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int len = first.len;
    const int T = whole ? max(1, (len + kWindow - 1) / kWindow) : 1;        // items
    // rows of up to a window that are cut into chunks of a piece (chunk_tokens_of)
    static_assert(kSeg / (4 * HETIS_FINE_CHUNK_BELOW) <= kWindow, "these are one item");

    // bounded wait for a word in LDS
    auto wait_word = [&](const int *word, int v, unsigned error) {
#pragma unroll 1
        for (int spin = 0; spin < kSpinLimit; ++spin) {
            if (__builtin_amdgcn_readfirstlane(mail_load(word)) == v) return;
            __builtin_amdgcn_s_sleep(kPollSleep);
        }
        if (lane == 0) report_error(p.control, error);
    };

    if (wave == NW) {
        // ------------------------------------------------------------ merger
        const int64_t out_row = (int64_t)first.seq * p.n_q_heads + first.g * R;
        if (blockIdx.x == 0 && lane == 0)
            record_way(p.control, spread ? kModeSpread : kModeSegments, whole ? kWayTeamRows : kWayTeamItems);
        RowFold<D, R> y;                            // the row's own workgroup: fold so far
        if (len <= 0) {
            store_result<D, R>(y.y, kKindZero, out_row, p, lane);
            return;
        }
        const int j = first.t0 / kSeg, in_seg = first.t0 - j * kSeg;
        const int n_seg = min(kSeg, len - j * kSeg);                // tokens of the segment
        const int ct = chunk_tokens_of(n_seg, kWindow, kSeg), per_chunk = ct / kPiece;
        const int ns = (n_seg + ct - 1) >> __builtin_ctz(ct);
        const int n_pieces = (min(whole ? kSeg : kWindow, n_seg - in_seg) + kPiece - 1) / kPiece;
        const bool own = whole || len <= kWindow;                   // the row is this workgroup's alone
        if (per_chunk == 1 && own) {
            // a chunk a wave, and no more than those: the whole row
#pragma unroll 1
            for (int v = 0; v < n_pieces; ++v) {
                wait_word(full + v, kMailFull, kErrWriterWait);
                RowRegs<D, R> g;
                g.load(l.rows[v].o, l.rows[v].lse, lane);
                y.take_in(g, v);
            }
            y.store(out_row, ns, p, lane);
            return;
        }
        int c = in_seg >> __builtin_ctz(ct), added = 0;             // chunk in its segment
        typename Policy::State tot;
#pragma unroll 1
        for (int v = 0; v < n_pieces; ++v) {
            const int slot = v / NW % 2, from = v % NW;
            wait_word(full + slot * NW + from, kMailFull, kErrWriterWait);
            typename Policy::State s;
            Policy::collect(s, l.state[slot][from], lane);
            if (v % per_chunk == 0) Policy::reset(tot);
            Policy::fold(tot, s);
            mail_store(full + slot * NW + from, kMailEmpty);
            if (v % per_chunk != per_chunk - 1 && v != n_pieces - 1) continue;
            Policy::finish(tot, l.o, l.lse, lane);
            wave_lds_fence();
            RowRegs<D, R> g;
            g.load(l.o, l.lse, lane);
            wave_lds_fence();
            if (!own) {
                store_partial_coherent<D, R>(g, (int64_t)first.row * p.max_segs + j * gc + c, p, lane, true);
                ++added;
            } else {
                y.take_in(g, c);
            }
            ++c;
        }
        if (own) {
            y.store(out_row, ns, p, lane);
        } else {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);                          // the chunk results are stored
            const int dest = first.row * p.max_segs + j * gc;
            unsigned before = 0;
            if (lane == 0)
                before = __hip_atomic_fetch_add(p.arrivals + arrival_counter<R>(p, dest, true, n_rows), (unsigned)added,
                                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            combine_if_last<D, R>(p, __builtin_amdgcn_readfirstlane((int)before), added, dest, ns, out_row, len, true,
                                  n_rows, lane);
        }
        return;
    }

    // ---------------------------------------------------------------- streaming waves
    TeamItem mine = first;
    mine.t0 += wave * kPiece;
    run_pieces<Policy, PAIRS>(p, mine, T, kWindow, l.staging[wave], lane, [&](typename Policy::State &st, int t) {
        if (len <= kSeg / (4 * HETIS_FINE_CHUNK_BELOW)) {           // a chunk of its own
            typename Policy::State tot;
            Policy::reset(tot);
            Policy::fold(tot, st);
            Policy::finish(tot, l.rows[wave].o, l.rows[wave].lse, lane);
            mail_store(full + wave, kMailFull);
            return;
        }
        int *flag = full + t % 2 * NW + wave;
        wait_word(flag, kMailEmpty, kErrMailboxWait);
        Policy::deposit(st, l.state[t % 2][wave], lane);
        mail_store(flag, kMailFull);
    });
}

}  // namespace hetis
