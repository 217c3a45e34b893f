// Launches of short rows: a wave a row, a workgroup a wave.
//
// What the persistent kernel does ahead of the first tile (lengths of all rows, tables, tickets, the pool) and
// behind the last (mailboxes, the writer wave's folds) pays where a row keeps a workgroup busy.  A row of a few tiles is
// over before: 640 rows of 64 tokens (r = 1) read 21 MB in 18 us.  Here a wave has its row's number from its
// workgroup's, asks for length, block ids and tiles, folds its pieces and chunks in registers, in the order and with
// the operations of the other launches, and stores the row; the hardware hands out the rows, and nothing is
// shared between waves.  Bound by HBM with many rows, by the chain length -> ids -> tiles -> fold with few.
// Workgroups of one wave: with four, a workgroup's place is taken by its longest row, and the launch ends
// unevenly (1280 rows of 128 to 256 tokens 28.2 us, two waves 24.5, one 23.8; 512 of 64 with r = 8 7.6, 6.5, 6.5).
// Times before and after, us: 640 rows of 64 tokens (r = 1) 17.8 -> 6.3, 264 of 32 to 256 17.9 -> 11.0; 512 of 64
// to 512 (r = 8, 64 dims) 18.9 -> 16.5; 2400 of 20 to 200 (64 dims) 35.4 -> 16.4; 2040 of 64 to 512 46.5 -> 28.9.
#pragma once
#include "attn_team.hpp"

namespace hetis {

// Whether a launch of `rows` rows on `cus` compute units, of up to `tokens` tokens each (what a row of the block
// table holds), goes this way.  The persistent kernel is the better one with rows of several hundred tokens, whose
// order it chooses (longest first) and whose chunks it spreads over the waves of a workgroup.  Both ways, us (the
// persistent kernel -> a wave a row; 1896 launches of both dims, every r and lengths up to `tokens` from an
// eighth, a half and seven eighths of it on are in profiles/wave_rows_lines.txt): inside the lines a wave a row is up
// to 2.6 times as fast and, but for one launch of 5 us, nowhere more than 2 % slower.
//  - no more rows than workgroups: a piece, which leaves the waves of a team nothing to share and saves the wait for
//    the fifth one (256 rows of up to 64 tokens, r = 1 5.4 -> 4.8, r = 2 6.5 -> 5.5, of up to 128 6.4 -> 6.8 and 7.2 ->
//    8.6; r = 8, of up to 128 7.7 -> 7.1, of up to 192 8.5 -> 9.7; r = 4, 64 dims 6.8 -> 5.5, of up to 192 7.5 -> 7.5).
//  - fewer than kMaxQuickRows: a full chunk, beyond which single chunks may be handed out, or two rows in a
//    workgroup's turn (264 rows of up to 256, r = 1 17.9 -> 11.0, of up to 384 12.4 -> 15.2; of up to 512, r = 8 22.2 ->
//    19.0, r = 4 21.7 -> 18.7, of up to 640 20.2 -> 23.0 and 19.1 -> 22.4).  With one or two query rows and close to
//    kMaxQuickRows the line lies further out (504 rows of 448 to 512, r = 1 27.7 -> 24.0; of 64 to 512 20.7 -> 21.7).
//  - up to 8 rows a compute unit: 512 tokens, which is right for 128 dims (512 rows of 64 to 512, r = 1 22.7 -> 21.4, r = 4
//    22.8 -> 20.7; of 80 to 640 24.3 -> 25.8, 1032 with r = 4 43.4 -> 45.1); with two query rows and less than a row for
//    every SIMD 384 (512 of 48 to 384 21.0 -> 20.6, of 64 to 512 25.1 -> 26.4).  With 64 dims a token costs half as
//    much and the line could lie further out: 2040 rows of 80 to 640 tokens, r = 1, are 1.36 times as fast, 520 with r = 8
//    (whose line is the one of two query rows) and 512 tokens 1.5 times.
//  - more: 384 (2096 rows of 448 to 512, r = 2 91.0 -> 98.3, of 336 to 384 72.7 -> 74.2; r = 1, of 256 to 512 73.8 ->
//    74.0).  Again not with 64 dims (5120 rows of 64 to 512, r = 1 92.8 -> 67.6).
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
