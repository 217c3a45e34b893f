// Launches of short rows: a wave a row, a workgroup a wave.
//
// What the persistent kernel does ahead of the first tile (lengths of all rows, tables, tickets, the pool) and
// behind the last (mailboxes, the writer wave's folds) pays where a row keeps a workgroup busy.  A row of a few tiles is
// over before: 640 rows of 64 tokens (r = 1) read 42 MB in 18 us.  Here a wave has its row's number from its
// workgroup's, asks for length, block ids and tiles, folds its pieces and chunks in registers, in the order and with
// the operations of the other launches, and stores the row; the hardware hands out the rows, and nothing is
// shared between waves.  Bound by HBM with many rows, by the chain length -> ids -> tiles -> fold with few.
// Workgroups of one wave: with four, a workgroup's place is taken by its longest row, and the launch ends
// unevenly (1280 rows of 128 to 256 tokens 28.2 us, two waves 24.5, one 23.8; 512 of 64 with r = 8 7.6, 6.5, 6.5).
// Times before and after, us: 640 rows of 64 tokens (r = 1) 18.0 -> 6.7, of 128 to 256 26.8 -> 14.3; 2560 of 128 to
// 256 56.5 -> 44.3; 512 of 64 (r = 8) 21.9 -> 6.5, 1024 of 128 to 256 35.8 -> 19.5, 2048 of 100 to 256 46.3 -> 35.7; 768
// of 10 to 40 (64 dims) 15.8 -> 4.8; 5120 of 10 to 90 37.9 -> 24.8.
#pragma once
#include "attn_team.hpp"

namespace hetis {

// Whether a launch of `rows` rows on `cus` compute units, of up to `tokens` tokens each (what a row of the block
// table holds), goes this way.  The persistent kernel is the better one with rows of several hundred tokens, whose
// order it chooses (longest first) and whose chunks it spreads over the waves of a workgroup:
//  - no more rows than workgroups: a piece, which leaves the waves of a team nothing to share and saves the wait for
//    the fifth one (16 rows of 16 to 64 tokens, r = 1 5.5 -> 5.1 us, r = 2 6.3 -> 5.1; 192 of 40 to 128, r = 8 7.5 -> 6.7;
//    rows of two pieces, r = 1 5.4 -> 5.8, r = 2 6.5 -> 8.1).  Fewer than kMaxQuickRows: a full chunk, beyond which
//    single chunks may be handed out (496 rows of 150 to 512, r = 8 25.8 -> 21.4 us, 272 27.8 -> 19.2).
//  - up to 8 rows a compute unit: 512 tokens (r = 1, 520 rows of 100 to 512 25.6 -> 21.5 us, 1280 of 384 to 512 54.9 ->
//    48.5; r = 8, 512 of 384 to 512 35.6 -> 23.3; of up to 768 tokens 30.4 -> 31.3, 28.9 -> 30.8 with r = 1, 22.5 ->
//    24.7 with 4 x 64).  Where a token costs a wave most for its bytes, two query rows or 8 of 64 dims, and there is
//    less than a row for every SIMD, 384 (512 rows of 100 to 512, r = 2 25.9 -> 27.7, 8 x 64 18.9 -> 19.8; of 100
//    to 384 21.1 -> 21.2 and 16.6 -> 15.8).
//  - more: 384 (3200 rows of 100 to 384 75.1 -> 67.6; of 384 to 512 120.5 -> 122.4, 5120 of 256 to 512 159.7 -> 162.7).
template <int D, int R>
constexpr bool row_a_wave(int64_t rows, int64_t cus, int64_t tokens)
{
    if (rows <= cus) return tokens <= decode_piece_tokens(R);
    if (rows < kMaxQuickRows) return tokens <= (R < 4 ? 256 : 512);
    constexpr bool slow = R == 2 || (R == 8 && D == 64);
    return tokens <= (rows > 8 * cus || (slow && rows < 4 * cus) ? 384 : 512);
}

template <class Policy, bool PAIRS>
__global__ __launch_bounds__(64, 2) void attn_wave_rows_kernel(const AttnParams p)
{
    constexpr int D = Policy::D, R = Policy::R;
    constexpr int kPiece = decode_piece_tokens(R);
    __shared__ struct alignas(16) {
        float o[R][D], lse[R];          // rows of a chunk on their way into registers of another layout
        unsigned char staging[Policy::kWaveLdsBytes ? Policy::kWaveLdsBytes : 16];
    } l;
    const int lane = threadIdx.x;
    if (blockIdx.x == 0 && lane == 0) record_way(p.control, kModeSegments, kWayWaveRows);
    TeamItem it;
    it.row = (int)blockIdx.x;
    it.b = PAIRS ? it.row : udiv(it.row, p.n_sel);
    it.seq = PAIRS ? uniform(p.pair_seq[it.b]) : it.b;
    it.g = PAIRS ? uniform(p.pair_head[it.b]) : uniform(p.head_ids[it.row - it.b * p.n_sel]);
    it.len = uniform(p.seq_lens[it.seq]);
    it.t0 = 0;
    const int64_t out_row = (int64_t)it.seq * p.n_q_heads + it.g * R;
    RowFold<D, R> fold;
    if (it.len <= 0) {
        store_result<D, R>(fold.y, kKindZero, out_row, p, lane);
        return;
    }
    const int n_pieces = (it.len + kPiece - 1) / kPiece;
    const int per_chunk = chunk_tokens_of(it.len, decode_chunk_tokens(R), decode_seg_tokens(R)) / kPiece;
    typename Policy::State tot;
    Policy::reset(tot);
    int c = 0;
    run_pieces<Policy, PAIRS>(p, it, n_pieces, kPiece, l.staging, lane, [&](typename Policy::State &st, int t) {
        Policy::fold(tot, st);
        if ((t + 1) % per_chunk != 0 && t != n_pieces - 1) return;
        Policy::finish(tot, l.o, l.lse, lane);
        wave_lds_fence();
        RowRegs<D, R> g;
        g.load(l.o, l.lse, lane);
        wave_lds_fence();
        fold.take_in(g, c++);
        Policy::reset(tot);
    });
    fold.store(out_row, c, p, lane);
}

}  // namespace hetis
