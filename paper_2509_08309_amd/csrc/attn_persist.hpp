// Persistent kernel of head-subset decode Attention: work enumeration, tile streaming and
// the combination of chunk results for Eq. (2b), independent of how a tile is turned into
// scores and sums (that is the Policy: vector ALU arithmetic for small query groups, MFMA
// for grouped-query attention).
//
// Units of work.  A ROW is one (enumeration row, selected KV head): a sequence (or, in pairs
// mode, a (sequence, head) pair) and one of the heads computed for it.  The tokens of a row
// are cut into SEGMENTS of seg_tokens tokens from token 0; a segment is cut into CHUNKS of
// chunk_tokens tokens.  A chunk is processed by ONE wave; a segment is processed by ONE
// workgroup, whose waves take its chunks and whose writer wave folds the chunk results
// together in LDS, in ascending chunk order, so a segment leaves the workgroup as a single
// result: the finished fp16 row when the segment is the whole row, an fp32 partial result
// (normalised sum and log-sum-exp) otherwise.  With seg_tokens = chunk_tokens every chunk is
// its own segment (the split-KV entry points); with seg_tokens = 4096 a row of up to 4096
// tokens never touches global memory between its first tile and its output row.
//
// Work enumeration: every workgroup loads the row lengths and builds two tables in LDS: the
// running count of whole segments per row, and the list of the rows that end in a shorter
// segment, sorted by the size class of that segment (kClasses classes, a counting sort done by
// the whole workgroup: see the prologue).  A flat segment number then decodes into (row,
// segment, head): whole segments first (binary search in the running counts), then the shorter
// ones from the largest class to the smallest (a look-up in the sorted list), so the segments
// handed out last are the short ones, which keeps the end of the launch short.
// Work distribution: segment number blockIdx.x belongs to the workgroup without asking (when
// every segment is a single chunk: two per streaming wave); the rest are tickets
// from a device counter, drawn by the workgroup's writer wave, which decodes a segment,
// reserves a fold slot for it and puts its chunks, ready to use, into an LDS pool; the
// streaming waves take chunks from the pool with an LDS atomic shortly before they finish the
// chunk at hand.  Which wave or workgroup computes a chunk has no influence on the arithmetic:
// a row's result is a function of its length and the compile-time constants alone.
// The ticket counter and a counter of workgroups that will draw no more are control words of
// the call's workspace (AttnParams::control); the last workgroup to count itself out sets both
// back to zero for the next launch.
// Scheduling modes (AttnParams::mode).  kModeSegments is the above.  kModeSplit: seg_tokens =
// chunk_tokens, every chunk leaves as a partial result for a separate merge launch.
// kModeSpread is an offer of the host for launches of few rows, where whole segments can leave
// much of the chip without work.  If there is no more than one full chunk of work for a workgroup, or a
// row for each, the waves of a workgroup share it (attn_team.hpp).  If there is more and the kernel takes the
// offer up, the unit handed out is the chunk (full
// chunks of all rows first, then the shorter ones), chunk results go through the partial buffers
// in global memory, and the wave that stores the last chunk result of a segment folds that
// segment's chunks with the operations and in the order of the in-LDS fold (fold_coef /
// fold_weight / fold_elem are shared), so that the mode never shows in a result.  These launches
// are bound by latency, not by HBM: what they pay for is the enumeration ahead of the first load,
// a second turn of chunks on some waves while others idle, and the round trips of the
// combination after the last chunk.  Hence: no tables and one barrier (every wave enumerates
// in registers), one chunk a wave across all compute units with the short ones second, the last
// chunk of a wave stored and combined by that wave, and partial results loaded many at a time.
// Measured, before (tables, chunks in row order, the writer wave combining one load at a time, a
// step's store as a launch of its own) and now: 16 chats of 1088 tokens on average x 13 heads of
// 128 45.1 -> 26.6 us; two documents of 20k and 27k tokens x 8 heads 70.4 -> 38.4; step of 144 pairs
// of 8-head groups 58.2 -> 41.0.
// Pieces.  A chunk is computed in up to four pieces (decode_piece_tokens) with sums of their own, folded lane
// by lane in ascending order, so that a chunk gives the same bits whether one wave computes it or four.  A
// fold costs a wave 0.1 to 0.2 us a piece: nothing in launches of many rows, which wait for HBM (1664 rows of
// 1069 tokens, 768 of 2176 with 8 heads: within 0.5 %), 1 to 3 % in some of 100 to 500 rows, a wave a chunk (252 of
// 100 to 400 tokens, r = 2, 64 dims 12.0 -> 12.2; 400 of 300 to 1600 of 64 dims 28.4 -> 28.7), against 10 to 40 %
// gained where four waves share a chunk.  (The first piece's fold changes nothing, but taking its state over as
// it is takes as many instructions as that fold: 28 launches 1.132 times as fast as before pieces, not 1.136.)
//
// A workgroup is NW streaming waves plus one writer wave; after the prologue they never
// meet at a barrier.
//   - Streaming waves stream the tiles of their chunk through a register ring of
//     Policy::ring slots; a slot is refilled right after it has been consumed, so up to
//     so many tile pairs per wave are in flight, and the ring runs on into the first tiles of
//     the next chunk before the current one is finished off.  Every global load is issued
//     unconditionally (indices clamped, tiles that do not exist turned into zero-length
//     buffer descriptors), so the in-order load counter is known exactly at every wait.
//     These waves do not store to global memory while loads are in flight (only the last chunk
//     of a wave may be stored by the wave itself): on gfx9-class hardware loads and stores
//     share one counter that is in order only among loads, so a single pending store would
//     force every later wait to drain all loads.  A finished chunk (normalised rows and
//     their base-2 log-sum-exp) is handed over through one of the wave's two LDS mailboxes.
//   - The writer wave polls the mailboxes.  A chunk that is a whole segment goes straight to
//     global memory (fp16 row, fp32 partial, or zeros for an empty sequence).  A chunk of a
//     longer segment is folded into the segment's slot: running maximum M, weight sum W and
//     weighted sum A with  M' = max(M, lse_c), A' = A 2^(M-M') + o_c 2^(lse_c-M'), W likewise;
//     chunk c is folded only after chunks 0..c-1 (a mailbox whose turn has not come stays
//     full), so the order of the floating-point operations is fixed.  After the last chunk
//     A / W leaves as the segment's result.
// Mailbox protocol (flag is a workgroup-scope atomic in LDS): EMPTY -> the producer fills
// data and header -> FULL -> the writer consumes it -> EMPTY.  A producer that has no more
// chunks marks its next mailbox DONE; the writer leaves when all NW are DONE.
// No wait can last for ever: chunks enter the pool in order, a wave's two mailboxes hold
// only chunks it took earlier, so the earliest chunk not yet folded can always be deposited
// and is always next in its segment.  All the same every wait is a polling loop with an
// iteration bound, so that every wave reaches its end whatever happens; a wait that runs
// into its bound sets a flag in the workspace's error word, which the host reads with
// hetis_attn_workspace_status (the launch may then have lost a result).
// Dynamic LDS: int lens[rows], int firstF[rows + 1] (and two spare words), uint16 order[rows],
// uint16 place[rows], int hids[n_sel] (pairs mode: hids[rows], pseq[rows]); NW x 2 mailboxes; fold
// slots; NW per-wave staging areas of Policy::kWaveLdsBytes.  Static LDS: the chunk pool and the
// scan array of the enumeration.
// Decode step with the store folded in (AttnParams::k_new): the new token's K and V rows go
// to position L - 1 of the cache inside this launch.  The writer wave stores the rows of a
// (sequence, head) right before it puts the chunk that contains position L - 1 into the pool,
// and waits for the stores to complete; the wave that takes the chunk runs on the same
// compute unit and takes it with an acquire, so it reads the new rows.  That chunk is never
// one of those taken without the pool, except in launches of few rows, where a streaming wave
// whose first chunk it is stores the rows itself before its first load (a store as a launch of its
// own ahead of these cost them 4.7 us and the gap between two launches).
// Pairs mode (per-request head subsets, Section 4.2 / 5.2.1): the rows of the enumeration are
// (sequence, KV head) pairs instead of sequences, each with its own block-table row over a
// pool of single-head tiles; everything else, the arithmetic included, is shared.
#pragma once
#include "attn_combine.hpp"
#include "attn_team.hpp"

namespace hetis {

// Size classes of a row's last, shorter segment, largest first: fifteen of one sixteenth of a
// whole segment each, then the last sixteenth split at 1/32, 1/64 and 1/128 of a segment.
constexpr int kLinClasses = 15;
constexpr int kClasses = kLinClasses + 4;
static_assert(kClasses + 1 <= 32, "class number + 1 is packed into five bits");
constexpr int kMaxSegChunks = 32;       // chunks of a segment, at most (one writer lane each)
constexpr int kPoolSize = 2 * kMaxSegChunks;   // chunk descriptors the LDS pool can hold
constexpr int kTicketBatch = 8;         // tickets per device atomic while segments are single chunks
// Chunks of multi-chunk segments a workgroup keeps waiting in its pool before it draws the
// next segment.
#ifndef HETIS_POOL_AHEAD
#define HETIS_POOL_AHEAD 2
#endif
// ... until so many segments are left to draw, in quarters of the number of workgroups.
#ifndef HETIS_LATE_SEGMENTS_X4
#define HETIS_LATE_SEGMENTS_X4 2
#endif
// Launches of up to this many segments a workgroup give every workgroup up to three segments
// without a ticket (0: one, always).
#ifndef HETIS_STATIC_SECOND_UPTO
#define HETIS_STATIC_SECOND_UPTO 4
#endif
// ... and only when the longest segment holds at most this many sixteenths of the tokens a
// workgroup gets on average.
#ifndef HETIS_STATIC_FLAT_X16
#define HETIS_STATIC_FLAT_X16 14
#endif
// A chunk, decoded: what a streaming wave needs to start on it and to label its result.
struct ChunkDesc {
    int b, g, seq;      // enumeration row (sequence, or pair), KV head, sequence of q / out rows
    int t0;             // first token of the chunk in its sequence, or of its last block in the table
    int n_tok;          // tokens of the chunk
    int n_ids;          // its entries of the block table, one or more, or 0: no work is left, the wave may finish
    int kind;           // kKindOut / kKindPartial / kKindZero (whole segment) or kKindFold
    int dest;           // Out / Zero: first of the R rows in `out`; Partial: slot in the partial
                        // buffers; Fold: the segment's fold slot
    int cs;             // Fold: index of the chunk in its segment
    int nseg;           // segments of the chunk's row
    int out_row;        // first of the R rows of the chunk's (sequence, head) in `out`
    int len;            // tokens of the chunk's row
};

// Chunks waiting to be taken by the streaming waves of one workgroup, in order.
struct ChunkPool {
    int next;                   // entries taken so far  (LDS atomic, streaming waves)
    int end;                    // entries published so far (written by the writer wave)
    ChunkDesc desc[kPoolSize];  // ring: entry i lives in desc[i % kPoolSize]
};

// One finished chunk on its way to the writer wave.
template <int D, int R>
struct alignas(16) Mailbox {
    float o[R][D];      // normalised output rows
    int kind, dest, cs, nseg;   // as in the chunk's descriptor (the first four read together)
    int out_row, len;
    int flag;           // kMailEmpty / kMailFull / kMailDone
    float lse[R];       // base-2 log-sum-exp of each row: m + log2(sum_t 2^(s_t - m))
};

// Running combination of the chunks of one segment (writer wave only).
template <int D, int R>
struct alignas(16) FoldSlot {
    float acc[R][D];    // sum over folded chunks of o_c 2^(lse_c - M)
    int next;           // chunk to fold next
    int ns;             // chunks of the segment
    int kind, dest;     // where the finished segment goes: kKindOut / kKindPartial
    float M[R];         // running maximum of lse_c (base 2)
    float W[R];         // sum over folded chunks of 2^(lse_c - M)
};

template <int R>
__host__ __device__ constexpr int fold_slots() { return R >= 4 ? 5 : 8; }

// Partial results (of segments, or in kModeSpread of chunks) that a writer wave has stored in
// one pass over its mailboxes and that still have to be counted in.  Ordering across waves and
// XCDs without cache-wide write-backs or invalidations (which were measured to cost several
// times the merge launch they replace): the partial results are written with device-coherent
// stores; the wave waits once until all its stores have completed, then bumps the counters of
// the rows concerned with device-scope atomics, one lane per result; the wave whose atomic
// completes a row reads the partial results with device-coherent loads issued after that
// atomic has returned, combines them into `out` and rearms the counter.  Waiting once per pass
// instead of once per result matters: a store takes a few microseconds to complete, about as
// long as the streaming waves of a workgroup need to produce the next results.
template <int NW>
struct Arrivals {
    int dest[NW], parts[NW], out_row[NW], len[NW];     // lives in LDS, used by the writer wave only
};

template <int D, int R, int NW>
__device__ __forceinline__ void count_in_and_combine(const AttnParams &p, const Arrivals<NW> &arr,
                                                     int n_arr, bool spread, int n_rows, int lane)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);                   // every store of this wave has completed
    unsigned old = 0;
    if (lane < n_arr)
        old = __hip_atomic_fetch_add(p.arrivals + arrival_counter<R>(p, arr.dest[lane], spread, n_rows), 1u,
                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll 1
    for (int i = 0; i < n_arr; ++i)
        combine_if_last<D, R>(p, __builtin_amdgcn_readlane((int)old, i), 1,
                              __builtin_amdgcn_readfirstlane(arr.dest[i]),
                              __builtin_amdgcn_readfirstlane(arr.parts[i]),
                              __builtin_amdgcn_readfirstlane(arr.out_row[i]),
                              __builtin_amdgcn_readfirstlane(arr.len[i]), spread, n_rows, lane);
}

struct ItemHdr {
    int b, g, seq;  // enumeration row (sequence, or pair), KV head, sequence of q / out rows
    int n_tok;      // tokens of this chunk
    int t0;         // first token of the chunk
    int kind, dest, cs;
    int nseg, out_row, len;
};

// Table bytes: lens, firstF (int), order and place (uint16), then the selected heads, or in pairs
// mode the head and the sequence of every pair.
__host__ __device__ constexpr size_t persist_table_bytes(int rows, int n_sel, bool pairs)
{
    return align16((size_t)(2 * rows + 2) * sizeof(int)) +
           align16((size_t)(2 * rows) * sizeof(unsigned short)) +
           align16((size_t)(pairs ? 2 * rows : n_sel) * sizeof(int));
}
// Rows of one launch, at most: bounds the static LDS of the enumeration (groups of 64 rows).
constexpr int kMaxRows = 2048;
constexpr int kMaxRowGroups = kMaxRows / 64;

template <class Policy, int NW>
__host__ __device__ constexpr size_t persist_lds_bytes(int rows, int n_sel, bool pairs)
{
    return persist_table_bytes(rows, n_sel, pairs) +
           2 * NW * sizeof(Mailbox<Policy::D, Policy::R>) +
           fold_slots<Policy::R>() * sizeof(FoldSlot<Policy::D, Policy::R>) +
           (size_t)NW * Policy::kWaveLdsBytes;
}

// Depth of the ring of tiles in a decode call of `rows` rows; `short_rows`: how many of 64 rows picked
// evenly are short as short_row() has it.  The depth follows the rows of the launch alone, whatever
// variant (see below) the width of the block table asks for.
//  - Fewer than kMaxQuickRows rows: deep.  Waves run dry before the launch ends, and those at work need
//    more in flight each (Policy::ring has the figures).
//  - Many rows, most of them of a few more tiles than the shallow ring holds: deep.  A row is read in one
//    go only as far as the ring reaches; each turn beyond it waits for memory with little in flight
//    (shallow -> deep, in us: 2976 rows of 20 to 80 tokens, r = 1, 128 dims 32.0 -> 29.3, 5984 of 40 to
//    160 76.6 -> 73.7, 3000 pairs of 20 to 80, r = 2 56.9 -> 52.7, 6000 of 64 dims 79.0 -> 75.1; but
//    5984 rows of 100 to 300 117.0 -> 119.6, r = 2, 64 dims 102.8 -> 105.0, and, one tile each, 6000
//    pairs of up to 16 62.7 -> 68.3).
//  - Otherwise shallow.
template <class Policy>
__host__ __device__ constexpr bool short_row(int tokens)
{
    return tokens > Policy::ring(false) * kBlockTokens && tokens <= 8 * kBlockTokens;
}
template <class Policy>
__host__ __device__ constexpr bool deep_ring(int rows, int short_rows)
{
    return rows < kMaxQuickRows || short_rows >= 40;
}

// VARIANT selects what is compiled in besides the common path; code that a launch cannot reach
// still costs it (launches measured 0.5 to 1.5 % faster without each of the two parts):
//   kVariantPlain  many rows, none of which can leave partial results; the split-KV entry points
//   kVariantFew    also the fixed second and third segments of launches with few segments a
//                  workgroup
//   kVariantMerge  also partial results that are combined inside the launch
//                  (AttnParams::arrivals is set), and single-chunk scheduling
//   kVariantTeam   also teams (attn_team.hpp), whose code costs launches that cannot have one up to 1.4 %: it is a quarter
//                  of the kernel, and the way to the first tile leads past it (with it -> without: 280 rows of 300 to
//                  1200 tokens, r = 8, 35.0 -> 34.5 us, 480 of 1000 to 1300 of 64 dims, r = 2, 37.1 -> 36.7, 400 of
//                  300 to 1600 of 64 dims 29.0 -> 28.8)
enum : int { kVariantPlain = 0, kVariantFew = 1, kVariantMerge = 2, kVariantTeam = 3 };
// Of the two that combine partial results: teams have a row or an item a workgroup, and a row has one item or more.
__host__ __device__ constexpr int merge_variant(int mode, int64_t rows, int64_t workgroups)
{
    return mode == kModeSpread && rows <= workgroups ? kVariantTeam : kVariantMerge;
}
// Instantiations that hold the split-KV scheduling (kModeSplit), in the writer wave and in the
// streaming waves alike; the host refuses such a launch on any other.
__host__ __device__ constexpr bool holds_split(int variant, bool pairs) { return variant == kVariantPlain && !pairs; }
template <class Policy, int NW, bool PAIRS, int VARIANT>
__global__ __launch_bounds__((NW + 1) * 64)
    __attribute__((amdgpu_waves_per_eu(Policy::kWavesPerEu))) void attn_chunk_persistent_kernel(
        const AttnParams p, const int batch)
{
    constexpr int D = Policy::D;
    constexpr int R = Policy::R;
    constexpr bool MERGE = VARIANT >= kVariantMerge;
    constexpr bool TEAM = VARIANT == kVariantTeam;
    constexpr bool FEW = VARIANT >= kVariantFew;
    constexpr bool CAN_SPLIT = holds_split(VARIANT, PAIRS);
    constexpr int NT = (NW + 1) * 64;
    constexpr int kRowBytes = D * 2;
    constexpr int NS = fold_slots<R>();
    using Mail = Mailbox<D, R>;
    using Fold = FoldSlot<D, R>;
    using Tile = typename Policy::Tile;
    extern __shared__ __align__(16) unsigned char smem[];
    int *lens = reinterpret_cast<int *>(smem);
    int *firstF = lens + batch;               // whole segments before row b; one spare word after
    // rows that end in a shorter segment (or, empty, in the segment that writes zeros), sorted
    // by the size class of that segment, largest first
    unsigned short *order =
        reinterpret_cast<unsigned short *>(smem + align16((size_t)(2 * batch + 2) * sizeof(int)));
    unsigned short *place = order + batch;    // enumeration only: a row's class and rank in it
    // KV head of position si in head_ids / of pair b; pairs mode: then the sequence of pair b
    int *hids = reinterpret_cast<int *>(reinterpret_cast<unsigned char *>(order) +
                                        align16((size_t)(2 * batch) * sizeof(unsigned short)));
    int *pseq = hids + batch;
    const int n_sel = PAIRS ? 1 : p.n_sel;    // heads per enumeration row
    const int n_ids = PAIRS ? batch : p.n_sel;
    unsigned char *after_tables = smem + persist_table_bytes(batch, p.n_sel, PAIRS);
    __shared__ ChunkPool pool;
    __shared__ Arrivals<NW> arrivals;       // writer wave only
    Mail *mail = reinterpret_cast<Mail *>(after_tables);             // [NW][2]
    Fold *fold = reinterpret_cast<Fold *>(after_tables + 2 * NW * sizeof(Mail));
    unsigned char *staging = reinterpret_cast<unsigned char *>(fold + NS);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // MERGE: decode calls only, whose cut is fixed: with constants the divisions are
    // shifts.  Code on the way to the first load is executed once and comes from the instruction
    // cache's misses, so its length is what it costs.
    const int seg_tokens = MERGE ? decode_seg_tokens(R) : p.seg_tokens;
    const int chunk_tokens = MERGE ? decode_chunk_tokens(R) : p.chunk_tokens;
    constexpr int kSegChunks = decode_seg_tokens(R) / decode_chunk_tokens(R);
    const bool merging = MERGE && p.arrivals != nullptr;

    // ---- launches of few rows (p.mode == kModeSpread: fewer than kMaxQuickRows rows x heads).
    // Every wave loads all row lengths and works out in registers, without a barrier, how the
    // launch is handed out, and (streaming waves) its own first item.  One of four ways:
    //  - lone: no more rows than workgroups, no row longer than a segment, and spread_pays() (attn_combine.hpp) says
    //    no: workgroup w takes row w as a team.
    //  - team: spread_pays(), and no more items (windows of a full chunk) than workgroups: workgroup w takes item
    //    w as a team.  A wave's chain of tiles is a quarter of a chunk's, and the chunk's pieces meet in LDS.
    //    With more items than workgroups the waves are busy with a chunk each, and a team has several
    //    items, one after the other, and its results pass through one wave: 16 rows of 2000 tokens (r =
    //    1, 128 items) 13.5 as chunks -> 10.4 us as teams, 64 rows of 500 to 3000 (r = 8, 220) 25.4 -> 18.7, 64
    //    of 300 to 1200 (r = 4, 64 dims) 16.6 -> 12.3; but 80 pairs of 850 (305 items) 15.3 -> 16.4, 64 rows of
    //    500 to 1500 (290) 14.9 -> 16.4, 300 of 300 to 1200 (980) 26.9 -> 32.6.  Rows whole: 230 of 600
    //    tokens 18.3 -> 15.9, 255 of 4096 88.3 -> 86.1, 240 of 1000 of 64 dims 20.1 -> 15.7, 256 of 300 to 900 (r =
    //    8, 64 dims) 17.3 -> 13.8, 16 of 17 to 255 of 64 dims 9.4 -> 5.5; 250 of 1000 to 4000 (r = 8) 68.0 -> 68.6.
    //  - spread: single chunks (see the top), when some row has more than one full chunk and
    //    spread_pays() says so.
    //  - otherwise whole segments through the tables, as in every other launch.
    // The tables cost 3 us of latency (scans over the workgroup, four barriers): a third of what
    // a launch of a few short rows takes.
    constexpr int QG = kMaxQuickRows / 64;
    bool spread = false;
    int q_len[MERGE ? QG : 1], q_seq[MERGE ? QG : 1], q_head[MERGE ? QG : 1];   // lane l: row 64 u + l
    int qA[MERGE ? QG : 1], qB[MERGE ? QG : 1];     // spread: full / other chunks before the row
    int totalA = 0, totalB = 0;
    auto full_chunks = [&](int L, int *others) {    // chunks of chunk_tokens tokens; shorter ones
        if (L <= 0) {
            *others = 1;                            // writes zeros
            return 0;
        }
        const int nF = udiv(L, seg_tokens), rt = L - nF * seg_tokens;
        const int ct = chunk_tokens_of(rt, chunk_tokens, seg_tokens);
        const int n = udiv(rt + ct - 1, ct), whole = ct == chunk_tokens ? udiv(rt, ct) : 0;
        *others = n - whole;
        return nF * kSegChunks + whole;
    };
    // value of enumeration row b (the same in all lanes) from the registers of the wave
    auto of_row = [&](const int (&q)[MERGE ? QG : 1], int b) {
        int x = 0;
#pragma unroll
        for (int u = 0; u < (MERGE ? QG : 1); ++u)
            if ((b >> 6) == u) x = __builtin_amdgcn_readlane(q[u], b & 63);
        return x;
    };
    int q_first_head = 0;                               // of the wave's first item
    // `batch`, to be compared with once more: the masks of the row groups, kept from one loop over them to the
    // next, take 32 scalar registers, and others are spilled for them
    auto rows_again = [&]() {
        int n = batch;
        asm volatile("" : "+s"(n));
        return n;
    };
    __shared__ int team_full[2 * NW];
    if (tid < 2 * NW) mail[tid].flag = team_full[tid] = kMailEmpty;
    if (tid == 0) {
        pool.next = 0;
        pool.end = 0;
    }
    if (MERGE && p.mode == kModeSpread) {
        // heads of the items this wave may start on: spread, team
        const int first_item = wave * (int)gridDim.x + (int)blockIdx.x;
        const int head_spread =
            PAIRS ? 0 : p.head_ids[first_item - (int)divide_by(first_item, p.sel_inverse) * n_sel];
        const int my_b = PAIRS ? (int)blockIdx.x : (int)divide_by(blockIdx.x, p.sel_inverse);
        const int my_si = (int)blockIdx.x - my_b * n_sel;
        const int head_team = PAIRS || !TEAM ? 0 : p.head_ids[my_si];
        // (groups beyond the launch's rows are branched over)
#pragma unroll
        for (int u = 0; u < QG; ++u) {
            q_len[u] = q_seq[u] = q_head[u] = qA[u] = qB[u] = 0;
            if (u * 64 >= batch) continue;
            const int i = min(u * 64 + lane, batch - 1);
            q_seq[u] = PAIRS ? p.pair_seq[i] : i;
            q_head[u] = PAIRS ? p.pair_head[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < QG; ++u)
            if (u * 64 < batch) q_len[u] = p.seq_lens[q_seq[u]];
        __syncthreads();                            // mailboxes and pool are ready
        int longest = 0, n_rows = rows_again();
        bool full_house = false;
#pragma unroll
        for (int u = 0; u < QG; ++u)
            if (u * 64 < n_rows) longest = max(longest, u * 64 + lane < n_rows ? q_len[u] : 0);
        longest = wave_max(longest);
        if (longest > seg_tokens) {
            // Rows of several segments: chunks while there are fewer segments than workgroups.  Two
            // rows of 20k and 27k tokens x 8 heads need it (see the top).  Around one segment a
            // workgroup neither way is always ahead: whole segments -> chunks, 20 rows of 15k to 60k,
            // r = 1 67 -> 72 us, r = 2 73 -> 78, r = 8 90 -> 85; 20 rows of 60k, r = 1 129 -> 110, r = 8
            // 154 -> 141; far beyond it whole segments are (500 rows of 5000, r = 2: 208 -> 234).
            int n_segments = 0;
            n_rows = rows_again();
#pragma unroll
            for (int u = 0; u < QG; ++u)
                if (u * 64 + lane < n_rows)
                    n_segments += max(1, udiv(max(q_len[u], 0) + seg_tokens - 1, seg_tokens));
            n_segments = __builtin_amdgcn_readlane(wave_scan_sum(n_segments), 63);
            spread = (long long)n_segments * n_sel < (long long)gridDim.x;
        } else if (longest > chunk_tokens) {
            // blocks and chunks of all rows, fewer than kMaxQuickRows, in one sum: below 2^17 and 2^14
            static_assert(kMaxQuickRows * kSegChunks <= 1 << 14 &&
                          kMaxQuickRows * (decode_seg_tokens(R) / kBlockTokens) <= 1 << 17, "sums fit");
            int sum = 0;
            n_rows = rows_again();
#pragma unroll
            for (int u = 0; u < QG; ++u) {
                if (u * 64 >= n_rows) continue;
                const int L = max(q_len[u], 1), ct = chunk_tokens_of(L, chunk_tokens, seg_tokens);
                const int sh = __builtin_ctz(ct);
                if (u * 64 + lane < n_rows)
                    sum += ((L + kBlockTokens - 1) / kBlockTokens << 14) + ((L + ct - 1) >> sh);
            }
            sum = __builtin_amdgcn_readlane(wave_scan_sum(sum), 63);
            const int tokens = (sum >> 14) * kBlockTokens * n_sel;
            spread = spread_pays<D, R, NW>((int)gridDim.x, batch * n_sel, longest, tokens,
                                           (sum & ((1 << 14) - 1)) * n_sel);
            // more than a full chunk a workgroup, whatever its rows
            full_house = tokens - batch * n_sel * (kBlockTokens - 1) > (int)gridDim.x * chunk_tokens;
        }
        const bool fits = TEAM && batch * n_sel <= (int)gridDim.x;          // a workgroup for each row
        const bool lone = fits && !spread && longest <= seg_tokens;
        // items (windows of a full chunk) of a row, and of all rows, per selected head
        auto items_of = [&](int L) { return max(1, (L + chunk_tokens - 1) / chunk_tokens); };
        int n_items = (int)gridDim.x + 1;
        // (counted only where the longest row's, with one for each other row, leave it open)
        if (fits && spread && !full_house &&
            (long long)(batch - 1 + items_of(longest)) * n_sel <= (long long)gridDim.x) {
            n_items = 0;
            n_rows = rows_again();
#pragma unroll
            for (int u = 0; u < QG; ++u)
                if (u * 64 + lane < n_rows) n_items += items_of(q_len[u]);
            n_items = __builtin_amdgcn_readlane(wave_scan_sum(n_items), 63);
        }
        const bool team = lone || (long long)n_items * n_sel <= (long long)gridDim.x;
        if (TEAM && __builtin_amdgcn_readfirstlane(team)) {
            if ((int)blockIdx.x >= (lone ? batch : n_items) * n_sel) return;
            int b = my_b, k = 0;
            const int si = my_si;
            if (!lone) {
                // the last row with no more than `left` items before it, group by group
                int left = b;
                b = 0;
                n_rows = rows_again();
#pragma unroll
                for (int u = 0; u < QG; ++u) {
                    if (u * 64 >= n_rows || b != u * 64) continue;
                    const int mine = u * 64 + lane < n_rows ? items_of(q_len[u]) : 0;
                    const int incl = wave_scan_sum(mine), all = __builtin_amdgcn_readlane(incl, 63);
                    if (left >= all) {
                        left -= all;
                        b += 64;
                    } else {
                        const int row = __builtin_popcountll(__builtin_amdgcn_ballot_w64(incl <= left));
                        b += row;
                        k = left - __builtin_amdgcn_readlane(incl - mine, row);
                        break;
                    }
                }
                b = __builtin_amdgcn_readfirstlane(b);
                k = __builtin_amdgcn_readfirstlane(k);
            }
            TeamItem it;
            it.b = b;
            it.seq = PAIRS ? __builtin_amdgcn_readfirstlane(of_row(q_seq, b)) : b;
            it.g = PAIRS ? __builtin_amdgcn_readfirstlane(of_row(q_head, b)) : head_team;
            it.row = b * n_sel + si;
            it.t0 = k * chunk_tokens;
            it.len = __builtin_amdgcn_readfirstlane(of_row(q_len, b));
            team_run<Policy, NW, PAIRS>(p, it, lone, spread, batch * n_sel, team_full, smem);
            return;
        }
        q_first_head = head_spread;
        if (spread) {
            n_rows = rows_again();
#pragma unroll
            for (int u = 0; u < QG; ++u) {
                if (u * 64 >= n_rows) continue;
                int nB = 0;
                int nA = full_chunks(q_len[u], &nB);
                if (u * 64 + lane >= n_rows) nA = nB = 0;
                const int inclA = wave_scan_sum(nA), inclB = wave_scan_sum(nB);
                qA[u] = totalA + inclA - nA;
                qB[u] = totalB + inclB - nB;
                totalA += __builtin_amdgcn_readlane(inclA, 63);
                totalB += __builtin_amdgcn_readlane(inclB, 63);
            }
        }
    }
    const bool quick = MERGE && spread;

    // ---- work enumeration.  Rows are handled in groups of 64 consecutive rows, one row a lane:
    // group u * (NW + 1) + wave belongs to round u of that wave, so a thread holds up to UR rows
    // in registers and one round covers a whole launch.
    //  1. All threads fetch the lengths of their rows (in pairs mode first the pair's sequence
    //     and head; the loads of all rounds are in flight together) and work out, per row, the
    //     number of whole segments and the size class of the last, shorter one.  Inside each
    //     group a DPP scan gives the running count of whole segments, and five ballots
    //     (one per bit of the class number) give every row the set of rows of its class, hence
    //     its rank among them and the class's count.
    //  2. The per-(class, group) counts, laid out class-major, and the per-group segment
    //     totals go through exclusive scans over the workgroup (three elements a thread, a
    //     DPP scan per wave, wave totals through LDS).
    //  3. Every thread writes its rows' table entries: firstF[row] = whole segments before
    //     the row; order[position] = row, position = rows of larger classes + rows of the
    //     same class in lower groups + rank.
    // size class of a last segment of `rt` tokens (0 < rt <= seg_tokens): 0 = the largest
    auto size_class = [&](int rt) {
        const int j = udiv(16 * rt - 1, seg_tokens);    // rt in (j/16, (j+1)/16] of a segment
        if (j >= 1) return kLinClasses - j;
        return kLinClasses + (rt <= (seg_tokens >> 5) ? 1 : 0) + (rt <= (seg_tokens >> 6) ? 1 : 0) +
               (rt <= (seg_tokens >> 7) ? 1 : 0);
    };
    constexpr int UR = (kMaxRows + NT - 1) / NT;        // rounds
    constexpr int kScanElems = kClasses * kMaxRowGroups + kMaxRowGroups;
    constexpr int E = (kScanElems + NT - 1) / NT;       // scan elements per thread
    __shared__ int scan[E * NT];                        // [class][group] counts, then [group] totals
    __shared__ int wave_tot[2 * (NW + 1)];
    const int n_groups = (batch + 63) / 64;
    if (!quick) {
        // The lengths go to LDS at once and the later steps run as loops that are not unrolled:
        // the prologue must not need more registers than the streaming loop, or the register
        // allocation of that loop suffers (measured: 12 % of the kernel's time).
        // Every load is issued unconditionally (indices clamped) and before the first use of any
        // of them, so that all of them are in flight together: a conditional load ends up
        // behind a branch and a full wait, and the prologue then pays one memory latency per
        // round instead of one in all (two in pairs mode).
        int row[UR], L[UR], head[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            const int i = min(tid + u * NT, batch - 1);
            row[u] = PAIRS ? p.pair_seq[i] : i;
            head[u] = PAIRS ? p.pair_head[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < UR; ++u) L[u] = p.seq_lens[row[u]];
        constexpr int UH = 4;                           // n_sel <= 1024 < UH * NT
        int sel[UH];
#pragma unroll
        for (int u = 0; u < UH; ++u) sel[u] = PAIRS ? 0 : p.head_ids[min(tid + u * NT, n_ids - 1)];
#pragma unroll
        for (int u = 0; u < UH; ++u)
            if (!PAIRS && tid + u * NT < n_ids) hids[tid + u * NT] = sel[u];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            const int i = tid + u * NT;
            if (i >= batch) continue;
            lens[i] = L[u];
            if (PAIRS) {
                hids[i] = head[u];
                pseq[i] = row[u];
            }
        }
    }
    if (!quick) {
    // Per row, kept until step 3: in its firstF entry the whole segments of the group's lower rows
    // (a word of its own: a split call over rows of 500k tokens in chunks of 16 has more than 2^21 in
    // a group), in its place entry (rank in its class) << 5 | (class + 1)
#pragma unroll 1
    for (int u = 0; u < UR; ++u) {
        const int i = tid + u * NT;
        const int g = u * (NW + 1) + wave;              // the row's group
        if (g >= n_groups) break;                       // same in all lanes: no rows from here on
        int nF = 0, cls = -1;
        if (i < batch) {
            const int L = lens[i];                      // this thread's own write
            nF = L > 0 ? udiv(L, seg_tokens) : 0;
            const int rt = L > 0 ? L - nF * seg_tokens : 0;
            if (rt > 0) cls = size_class(rt);
            if (L <= 0 && p.direct_single) cls = kClasses - 1;   // the segment that writes the zeros
        }
        const int incl = wave_scan_sum(nF);
        int rank = 0;
        // lanes of the same class, from one ballot per bit of the class number
        unsigned long long same = ~0ull;
#pragma unroll
        for (int bit = 0; bit < 5; ++bit) {
            const bool one = ((cls + 1) >> bit) & 1;
            const unsigned long long b = __builtin_amdgcn_ballot_w64(one);
            same &= one ? b : ~b;
        }
        rank = __builtin_amdgcn_mbcnt_hi((unsigned)(same >> 32),
                                         __builtin_amdgcn_mbcnt_lo((unsigned)same, 0));
        const int count = __builtin_popcountll(same);
        if (i < batch) {
            firstF[i] = incl - nF;
            place[i] = (unsigned short)((rank << 5) | (cls + 1));
        }
        // class counts of the group: zero, then the last row of every class present writes its own
        if (lane < kClasses) scan[lane * n_groups + g] = 0;
        wave_lds_fence();
        if (cls >= 0 && rank == count - 1) scan[cls * n_groups + g] = count;
        if (lane == 63) scan[kClasses * n_groups + g] = incl;
    }
    __syncthreads();
    {
        // exclusive scans of scan[0, n_cls) (class counts) and scan[n_cls, n_all) (segment totals)
        const int n_cls = kClasses * n_groups, n_all = n_cls + n_groups;
        int v[E], sumC = 0, sumF = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int idx = tid * E + e;
            v[e] = idx < n_all ? scan[idx] : 0;
            if (idx < n_cls)
                sumC += v[e];
            else
                sumF += v[e];
        }
        const int inclC = wave_scan_sum(sumC), inclF = wave_scan_sum(sumF);
        if (lane == 63) {
            wave_tot[wave] = inclC;
            wave_tot[NW + 1 + wave] = inclF;
        }
        __syncthreads();
        int baseC = inclC - sumC, baseF = inclF - sumF, allC = 0, allF = 0;
#pragma unroll
        for (int w = 0; w < NW + 1; ++w) {
            const int tc = wave_tot[w], tf = wave_tot[NW + 1 + w];
            if (w < wave) {
                baseC += tc;
                baseF += tf;
            }
            allC += tc;
            allF += tf;
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int idx = tid * E + e;
            if (idx < n_cls) {
                scan[idx] = baseC;
                baseC += v[e];
            } else if (idx < n_all) {
                scan[idx] = baseF;
                baseF += v[e];
            }
        }
        if (tid == 0) {
            firstF[batch] = allF;               // whole segments of all rows
            lens[2 * batch + 1] = allC;         // number of listed rows, kept in the table's spare word
        }
    }
    __syncthreads();
#pragma unroll 1
    for (int u = 0; u < UR; ++u) {
        const int i = tid + u * NT;
        const int g = u * (NW + 1) + wave;
        if (i >= batch) break;
        const int info = place[i];
        const int cls = (info & 31) - 1, rank = info >> 5;
        firstF[i] += scan[kClasses * n_groups + g];
        if (cls >= 0) order[scan[cls * n_groups + g] + rank] = (unsigned short)i;
    }
    __syncthreads();
    }
    const int totalF = quick ? 0 : firstF[batch];             // whole segments of all rows
    // segments (spread: chunks) of this launch
    const int total = (spread ? totalA + totalB : totalF + lens[2 * batch + 1]) * n_sel;
    if (spread && wave == NW) {
        // tables for the writer wave's own use: rows, and chunks before each row
#pragma unroll
        for (int u = 0; u < QG; ++u) {
            if (u * 64 >= batch) continue;
            const int i = u * 64 + lane;
            if (i >= batch) continue;
            lens[i] = q_len[u];
            firstF[i] = qA[u];
            scan[i] = qB[u];
            if (PAIRS) {
                hids[i] = q_head[u];
                pseq[i] = q_seq[u];
            }
        }
        if (!PAIRS)
            for (int i = lane; i < n_ids; i += 64) hids[i] = p.head_ids[i];
        wave_lds_fence();
    }

    // segment number -> (row, segment, head): whole segments come first (binary search in the
    // running counts), last segments after them by size class (sorted list).  Works per lane.
    auto upper = [&](const int *tab, int key) {               // last b with tab[b] <= key
        int lo = 0, hi = batch - 1;
#pragma unroll 1
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tab[mid] <= key)
                lo = mid;
            else
                hi = mid - 1;
        }
        return lo;
    };
    struct Segment {
        int b, g, seq;      // enumeration row, KV head, sequence
        int t0, n_tok;      // first token, tokens
        int ct, ns;         // tokens per chunk, chunks
        int kind, dest;     // where the whole segment goes
        int nseg, out_row;  // segments of the row (kModeSpread: its chunks); first of its R rows in `out`
        int tail;           // 1: the segment ends with the row's last token
        int len;            // tokens of the row
    };
    auto chunk_for = [&](int n_tok) { return chunk_tokens_of(n_tok, chunk_tokens, seg_tokens); };
    // kModeSpread: items are numbered full chunks of all rows first, then the shorter ones, heads
    // fastest; chunk k of those of row b is returned as a segment of one chunk
    auto spread_segment = [&](int b, int si, bool full, int k, int L, int g, int seq) {
        Segment s;
        constexpr int gc = kSegChunks;
        const int nF = L > 0 ? udiv(L, seg_tokens) : 0;
        const int rt = max(L, 0) - nF * seg_tokens;
        int j, c;
        s.ct = chunk_tokens;
        if (full) {
            j = udiv(k, gc);
            c = k - j * gc;
            s.n_tok = chunk_tokens;
        } else {
            j = nF;
            s.ct = chunk_for(rt);
            c = k + (s.ct == chunk_tokens ? udiv(rt, chunk_tokens) : 0);
            s.n_tok = max(0, min(s.ct, rt - c * s.ct));
        }
        s.t0 = j * seg_tokens + c * s.ct;
        s.ns = 1;
        s.b = b;
        s.g = g;
        s.seq = seq;
        s.nseg = nF * gc + udiv(rt + chunk_for(rt) - 1, chunk_for(rt));
        s.out_row = s.seq * p.n_q_heads + s.g * R;
        s.tail = L > 0 && s.t0 + s.n_tok == L;
        s.len = L;
        if (L <= 0) {
            s.kind = kKindZero;
            s.dest = s.out_row;
        } else if (s.nseg == 1) {
            s.kind = kKindOut;
            s.dest = s.out_row;
        } else {
            s.kind = kKindPartial;
            s.dest = (b * n_sel + si) * p.max_segs + j * gc + c;
        }
        return s;
    };
    auto decode_spread = [&](int itemno) {          // from the writer wave's tables, per lane
        const int w = min(itemno, max(total - 1, 0));
        const int cg = PAIRS ? w : w / n_sel;
        const int si = PAIRS ? 0 : w - cg * n_sel;
        const bool full = cg < totalA;
        const int key = full ? cg : cg - totalA;
        const int *tab = full ? firstF : scan;
        const int b = upper(tab, key);
        return spread_segment(b, si, full, key - tab[b], lens[b], hids[PAIRS ? b : si],
                              PAIRS ? pseq[b] : b);
    };
    // the wave's first item -> chunk, from the registers of the wave
    auto quick_spread = [&](int item) {
        const int cg = PAIRS ? item : (int)divide_by(item, p.sel_inverse);
        const int si = PAIRS ? 0 : item - cg * n_sel;
        const bool full = cg < totalA;
        const int key = full ? cg : cg - totalA;
        int b = -1;                                 // last row with no more than `key` before it
#pragma unroll
        for (int u = 0; u < (MERGE ? QG : 1); ++u)
            if (u * 64 < batch)
                b += __builtin_popcountll(__builtin_amdgcn_ballot_w64(
                    u * 64 + lane < batch && (full ? qA[u] : qB[u]) <= key));
        b = __builtin_amdgcn_readfirstlane(b);
        const int before = full ? of_row(qA, b) : of_row(qB, b);
        return spread_segment(b, si, full, key - before, of_row(q_len, b),
                              PAIRS ? of_row(q_head, b) : q_first_head, PAIRS ? of_row(q_seq, b) : b);
    };
    // what of a segment of row b follows from its length
    auto row_segment = [&](int b, int si, int j, int n_tok, int L, int g, int seq) {
        Segment s;
        s.b = b;
        s.n_tok = n_tok;
        s.t0 = j * seg_tokens;
        s.ct = chunk_for(s.n_tok);
        s.ns = max(1, udiv(s.n_tok + s.ct - 1, s.ct));
        s.g = g;
        s.seq = seq;
        const int n_segs = udiv(max(L, 0) + seg_tokens - 1, seg_tokens);
        s.nseg = n_segs;
        s.out_row = s.seq * p.n_q_heads + s.g * R;
        s.tail = L > 0 && s.t0 + s.n_tok == L;
        s.len = L;
        if (L <= 0) {
            s.kind = kKindZero;
            s.dest = s.out_row;
        } else if (p.direct_single && n_segs <= 1) {
            s.kind = kKindOut;
            s.dest = s.out_row;
        } else {
            s.kind = kKindPartial;
            s.dest = (s.b * n_sel + si) * p.max_segs + j;
        }
        return s;
    };
    auto decode = [&](int segno) {
        if (spread) return decode_spread(segno);
        const int w = min(segno, max(total - 1, 0));
        const int cg = PAIRS ? w : w / n_sel;
        const int si = PAIRS ? 0 : w - cg * n_sel;
        int b, L, j, n_tok;
        if (cg < totalF) {
            b = upper(firstF, cg);
            j = cg - firstF[b];
            L = lens[b];
            n_tok = seg_tokens;
        } else {
            b = order[cg - totalF];
            L = lens[b];
            j = L > 0 ? udiv(L, seg_tokens) : 0;
            n_tok = L > 0 ? L - j * seg_tokens : 0;
        }
        return row_segment(b, si, j, n_tok, L, hids[PAIRS ? b : si], PAIRS ? pseq[b] : b);
    };
    // chunk i of a segment; `slot`: the segment's fold slot (segments of several chunks)
    auto chunk_of = [&](const Segment &s, int i, int slot) {
        ChunkDesc d;
        d.b = s.b;
        d.g = s.g;
        d.seq = s.seq;
        // (a length past the block table, the caller's error, reads the row's last entry again, as in a team.
        // Bounded here: with the bounds where the ids are loaded the step of 145 pairs, r = 8, took 40.1 us
        // instead of 39.8, with one in each lane 240 rows of 1000 tokens of 64 dims 15.2 instead of 14.9.)
        d.t0 = min((s.t0 + i * s.ct) / kBlockTokens, p.max_blocks_per_seq - 1) * kBlockTokens;
        d.n_tok = max(0, min(s.ct, s.n_tok - i * s.ct));
        d.n_ids = max(1, min((d.n_tok + kBlockTokens - 1) / kBlockTokens, p.max_blocks_per_seq - d.t0 / kBlockTokens));
        d.kind = s.ns > 1 ? (int)kKindFold : s.kind;
        d.dest = s.ns > 1 ? slot : s.dest;
        d.cs = i;
        d.nseg = s.nseg;
        d.out_row = s.out_row;
        d.len = s.len;
        return d;
    };
    // Work a workgroup has without a ticket.  When segments have several chunks: segment number
    // blockIdx.x, whose first NW chunks the streaming waves take directly (wave v takes chunk
    // v) and which owns fold slot 0.  When every segment is a single chunk, two per streaming
    // wave v: kModeSplit: segments (blockIdx.x + k gridDim.x) * NW + v, k = 0, 1 (the waves of a
    // workgroup work on neighbouring heads of one chunk position).  kModeSpread: item
    // v gridDim.x + blockIdx.x, so that a launch of fewer items than waves works on every compute
    // unit, and, through the pool, the items that lie as far from the other end of the first
    // 2 NW gridDim.x (the shortest items come last: a wave with a full chunk gets a short one or
    // none).  Tickets number the segments after these.
    const bool split_mode = CAN_SPLIT && p.mode == kModeSplit;
    const bool single_mode = split_mode || spread;
    const bool have_first = (int)blockIdx.x < total;
    const bool step_mode = p.k_new != nullptr;      // never with kModeSplit
    // chunks of the first segment that are taken without the pool: the first NW.  When the new
    // token is stored in this launch, the one that holds the row's last position is left to the
    // pool, unless (launches of few rows) the streaming wave that takes it stores the rows itself.
    auto direct_chunks = [&](const Segment &s0) {
        int n = min(NW, s0.ns);
        if (!MERGE && step_mode && s0.tail && n == s0.ns) --n;
        return n;
    };
    // store of the new token's rows of the segment's (sequence, head), done before the chunk
    // that reads them becomes visible to the streaming waves.  Like a store on its own it leaves
    // out a row whose position is past its block table or whose head does not exist; a negative
    // block id only in the variant that serves launches of few rows: where every workgroup stores
    // many rows, a store that hangs on a loaded value costs 2 to 5 % (2400 rows of 125 to 500 tokens,
    // r = 2, 64 dims: 69.9 -> 73.4 us)
    auto store_tail = [&](const Segment &sg) {
        const int L = sg.t0 + sg.n_tok;             // tail segment: the row's length
        const int pos = L - 1;
        const int j = pos / kBlockTokens, n_kv_heads = p.n_q_heads / R;
        const int blk = p.block_table[(int64_t)sg.b * p.max_blocks_per_seq + min(j, p.max_blocks_per_seq - 1)];
        const bool inside = (j < p.max_blocks_per_seq) & ((unsigned)sg.g < (unsigned)n_kv_heads) &
                            (!MERGE | (blk >= 0));
        const int64_t off = (int64_t)blk * p.stride_block + (PAIRS ? 0 : (int64_t)sg.g * p.stride_head);
        store_new_rows<D>(p, sg.seq, sg.g, off, pos % kBlockTokens, n_kv_heads, lane, inside);
    };
    // the same by the streaming wave whose first chunk it is: nothing of it is in flight yet
    auto store_own_tail = [&](const Segment &sg) {
        store_tail(sg);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
    };
    if (wave == NW) {
        // ------------------------------------------------------------ writer wave
        // Segments a workgroup has without a ticket: its first, and, in some launches of at most
        // HETIS_STATIC_SECOND_UPTO segments a workgroup, a second and a third.  The second comes
        // from the other end of the next gridDim.x segments of the sorted list, so that the two
        // together hold about the same number of tokens in every workgroup; the third goes by
        // the rank of that sum (the largest sum takes the shortest of the following gridDim.x
        // segments).  With so few segments the draws of all workgroups come in bursts (every
        // pool runs low at the same moment) and pair long segments with long ones as often as
        // not; with many segments a workgroup the tickets even the load out by themselves, and
        // fixing more of it only takes room from them.  Three conditions besides the number of
        // segments.  The longest segment must be well below the tokens a workgroup gets on
        // average: where a few long rows stand out (their workgroups are what the launch waits
        // for), they must not be given more, and the tickets see to that.  The segments must
        // differ in length, or there is nothing to balance.  And beyond two segments a
        // workgroup the longest segment must have at least as many chunks as a workgroup has
        // streaming waves: shorter rows need no balancing, and the waves would wait for the
        // writer wave's sums and for the first draw behind them.
        // The segments that need no ticket wait in a queue of three numbers (q0 next; -1: none),
        // worked out here, before the loop, so that the loop itself carries no state for them.
        const int Gn = (int)gridDim.x;
        int n_fixed = Gn * (single_mode ? 2 * NW : 1);
        int q0 = have_first && !single_mode ? (int)blockIdx.x : -1, q1 = -1, q2 = -1;
        if (FEW && HETIS_STATIC_SECOND_UPTO > 0 && !single_mode && total > Gn &&
            (long long)total <= (long long)HETIS_STATIC_SECOND_UPTO * Gn) {
            // tokens of segment number `segno` (whole-segment scheduling): what decode() would
            // put into n_tok, without the rest of it
            auto seg_n_tok = [&](int segno) {
                const int w = min(segno, max(total - 1, 0));
                const int cg = PAIRS ? w : w / n_sel;
                if (cg < totalF) return seg_tokens;
                const int L = lens[order[cg - totalF]];
                return L > 0 ? L - udiv(L, seg_tokens) * seg_tokens : 0;
            };
            const int tok0 = seg_n_tok(0);
            const bool long_rows = udiv(tok0 + chunk_for(tok0) - 1, chunk_for(tok0)) >= NW;
            // tokens of the launch from the class counts (a class's rows taken at the middle of
            // its range; one class a lane, then a sum over the wave): the same sum of integers in
            // every workgroup
            const int listed = lens[2 * batch + 1];
            long long part = 0;
            if (lane < kClasses) {
                const int c = lane;
                const int first_c = scan[c * n_groups];
                const int next_c = c + 1 < kClasses ? scan[(c + 1) * n_groups] : listed;
                const int j = kLinClasses - c;                // classes of a sixteenth of a segment
                const int mid = c < kLinClasses ? (2 * j + 1) * seg_tokens / 32
                                                : (3 * seg_tokens) >> (c - kLinClasses + 6);
                part = (long long)(next_c - first_c) * mid;
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
            const long long mean_load = ((long long)totalF * seg_tokens + part) * n_sel / Gn;
            const bool flat = 16ll * tok0 <= (long long)HETIS_STATIC_FLAT_X16 * mean_load;
            // ... and there must be something to balance: with segments of (nearly) one size the
            // tickets do better, they give the last segments to the workgroups that run fastest
            const int tok_last = seg_n_tok(min(total, 3 * Gn) - 1);
            const bool uneven = 4ll * tok0 > 5ll * tok_last;
            if (flat && uneven && (total <= 2 * Gn || long_rows)) {
                n_fixed = 2 * Gn;
                const int second_no = 2 * Gn - 1 - (int)blockIdx.x;
                if (second_no < total) q1 = second_no;
                if (total > 2 * Gn) {
                    // The third: the workgroup whose first two hold the most tokens takes the
                    // shortest of the next Gn segments, and so on (rank among the sums, which
                    // every workgroup can work out for itself).
                    n_fixed = 3 * Gn;
                    auto two_sum = [&](int b) {
                        const int s2 = 2 * Gn - 1 - b;
                        return seg_n_tok(b) + (s2 < total ? seg_n_tok(s2) : 0);
                    };
                    const int my = __builtin_amdgcn_readfirstlane(two_sum((int)blockIdx.x));
                    int rank = 0;
#pragma unroll 1
                    for (int b0 = 0; b0 < Gn; b0 += 64) {
                        const int b = b0 + lane;
                        const int sum_b = two_sum(min(b, Gn - 1));
                        const bool larger =
                            b < Gn && (sum_b > my || (sum_b == my && b < (int)blockIdx.x));
                        rank += __builtin_popcountll(__builtin_amdgcn_ballot_w64(larger));
                    }
                    const int third_no = 3 * Gn - 1 - rank;
                    if (third_no < total) q2 = third_no;
                }
            }
        }
        unsigned boxes = 0;               // bit v: the mailbox of wave v that is read next
        int done_mask = 0;
        int idle = 0;
        int pool_end = 0;                 // entries published so far
        unsigned busy = 0;                // fold slots in use
        bool exhausted = total <= n_fixed;            // no segment left to draw
        // A workgroup that will draw no more tickets counts itself out at once, not when it
        // ends: the answer (was it the last one?) is needed only at the end, and by then the
        // atomic's round trip, which would otherwise be the last thing the kernel waits for,
        // is long over.  The last workgroup to count itself out rearms both counters; that is
        // safe while others still compute, since none of them draws again.  Where no workgroup
        // draws (the same numbers everywhere, so the same answer) nobody counts: 256 atomics on
        // one address take longer than a launch of one turn has left, wherever the writer wave
        // issues them (counted ahead of the first pass, behind its published work, and not at all:
        // 252 rows of 25 to 100 tokens, r = 4, 64 dims 9.2, 10.4 and 8.8 us; 64 rows of 300 to 1200
        // 17.6, 18.4 and 16.9; 508 of 500 to 2000 39.2, 40.1 and 38.1; r = 1, 62 rows of at most 35
        // tokens 7.9, 7.0 and 7.05; 96 pairs of up to 1300, 64 dims 13.7, 13.2 and 11.5).
        const bool draws = total > n_fixed;
        bool counted_out = !draws;
        unsigned gone_before = 0;                     // lane 0: workgroups counted out before this one
        // (The address passes for one that differs between lanes: of an atomic on one address the
        // compiler broadcasts the result at once, and the wave waited for it here, in launches of one
        // turn before the streaming waves had been told that there is no more work.)
        auto count_out = [&]() {
            int same = 0;
            asm volatile("" : "+v"(same));
            if (lane == 0)
                gone_before = __hip_atomic_fetch_add(p.control + kCtlGone + same, 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
            counted_out = true;
        };
        bool first = have_first && !single_mode;      // the next segment to publish is the workgroup's first
        bool closed = false;              // the "no work left" entries have been published
        // Segments drawn and decoded (one per lane, lanes [pend_i, pend_n) still to publish)
        Segment mine{};
        int pend_i = 0, pend_n = 0;
        long long last_base = n_fixed;    // number of the last segment drawn here
        int last_tok = seg_tokens;        // tokens of the last segment seen
        const long long wave_round = (long long)gridDim.x * NW;
        auto bcast = [&](const Segment &s, int k) {
            Segment r;
            r.b = __builtin_amdgcn_readlane(s.b, k);
            r.g = __builtin_amdgcn_readlane(s.g, k);
            r.seq = __builtin_amdgcn_readlane(s.seq, k);
            r.t0 = __builtin_amdgcn_readlane(s.t0, k);
            r.n_tok = __builtin_amdgcn_readlane(s.n_tok, k);
            r.ct = __builtin_amdgcn_readlane(s.ct, k);
            r.ns = __builtin_amdgcn_readlane(s.ns, k);
            r.kind = __builtin_amdgcn_readlane(s.kind, k);
            r.dest = __builtin_amdgcn_readlane(s.dest, k);
            r.nseg = __builtin_amdgcn_readlane(s.nseg, k);
            r.out_row = __builtin_amdgcn_readlane(s.out_row, k);
            r.tail = __builtin_amdgcn_readlane(s.tail, k);
            r.len = __builtin_amdgcn_readlane(s.len, k);
            return r;
        };
        bool own_items = spread;          // the workgroup's own items beyond its waves' first ones
        while (done_mask != (1 << NW) - 1 && idle < kSpinLimit) {
            bool progressed = false;
            // (Here and not behind the work that the pass before it published: 1472 rows of 40 to 160
            // tokens 27.4 us and 28.5, 6000 pairs of 20 to 80 83.4 and 85.1.)
            if (exhausted && !counted_out) count_out();
            // One look at everything the wave waits for: the pool's counter, and lane v at the flag of
            // wave v's next mailbox.
            const int taken_now = __hip_atomic_load(&pool.next, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            const int looked = min(lane, NW - 1);
            const int seen = mail_load(&mail[looked * 2 + (int)((boxes >> looked) & 1u)].flag);
            const int taken = __builtin_amdgcn_readfirstlane(taken_now);
            const int done_now = (int)__builtin_amdgcn_ballot_w64(lane < NW && seen == kMailDone);
            unsigned full = (unsigned)__builtin_amdgcn_ballot_w64(lane < NW && seen == kMailFull);
            if (done_now != done_mask) progressed = true;
            done_mask = done_now;
            // ---- keep the chunk pool ahead of the streaming waves
            // Draw.  Work parked in one workgroup's pool cannot be taken by another that has run
            // dry, so little is drawn at a time and late; but a same-address device atomic
            // costs about as much as a short chunk, so short segments are drawn several at a
            // time.  Every chunk its own segment (split-KV): batches that shrink as the work
            // runs out.  Otherwise: about one full chunk's worth of tokens per draw, judged by
            // the last segment seen (they come longest first), drawn when fewer than
            // HETIS_POOL_AHEAD chunks (one, near the end) or than a draw's worth are waiting.
            // (Only in a pass that can draw: the division leaves scratch registers behind that the
            // compiler takes to be still in use by the counting atomic above, and waits for it.)
            int n_draw = 0, ahead = 0;
            if (!exhausted && pend_i == pend_n) {
                const long long left = (long long)total - last_base;
                if (single_mode) {
                    n_draw = left > 8 * wave_round ? kTicketBatch : (left > 2 * wave_round ? 2 : 1);
                    ahead = n_draw;
                } else {
                    n_draw = max(1, min(kTicketBatch, chunk_tokens / max(last_tok, 1)));
                    ahead = max(4 * left > (long long)gridDim.x * HETIS_LATE_SEGMENTS_X4 ? HETIS_POOL_AHEAD : 1, n_draw);
                }
            }
            int want = -1;                // segment to decode in this pass (one a lane)
            if (MERGE && own_items) {
                want = (NW + lane) * Gn + Gn - 1 - (int)blockIdx.x;          // lanes 0 .. NW - 1
                pend_n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < NW && want < total));
                own_items = false;
                progressed = true;
            } else if (pend_i == pend_n && q0 >= 0) {
                // the next of the workgroup's own segments
                want = q0;
                q0 = q1;
                q1 = q2;
                q2 = -1;
                pend_i = 0;
                pend_n = 1;
                progressed = true;
            } else if (pend_i == pend_n && !exhausted && pool_end - taken < ahead) {
                unsigned t = 0;
                if (lane == 0)
                    t = __hip_atomic_fetch_add(p.control + kCtlTickets, (unsigned)n_draw,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const long long base = n_fixed + __builtin_amdgcn_readfirstlane(t);
                last_base = base;
                if (base + n_draw >= total) exhausted = true;
                pend_i = 0;
                pend_n = (int)max(0ll, min((long long)n_draw, (long long)total - base));
                if (pend_n > 0) want = (int)min(base + lane, (long long)total - 1);
                progressed = true;
            }
            if (want >= 0) mine = decode(want);
            if (pend_i < pend_n) {
                // all remaining drawn segments are single chunks: publish them together
                const bool single = __builtin_amdgcn_ballot_w64(lane >= pend_i && lane < pend_n &&
                                                                mine.ns != 1) == 0;
                if (single && !first) {
                    const int cnt = pend_n - pend_i;
                    if (pool_end + cnt - taken <= kPoolSize) {
                        if (step_mode) {
#pragma unroll 1
                            for (int e = pend_i; e < pend_n; ++e) {
                                const Segment sg = bcast(mine, e);
                                if (sg.tail) store_tail(sg);
                            }
                            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                            __builtin_amdgcn_s_waitcnt(0);
                        }
                        if (lane >= pend_i && lane < pend_n)
                            pool.desc[(pool_end + lane - pend_i) % kPoolSize] = chunk_of(mine, 0, 0);
                        pool_end += cnt;
                        __hip_atomic_store(&pool.end, pool_end, __ATOMIC_RELEASE,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                        last_tok = __builtin_amdgcn_readlane(mine.n_tok, pend_n - 1);
                        pend_i = pend_n;
                        progressed = true;
                    }
                } else {
                    const Segment seg = bcast(mine, pend_i);
                    if (pool_end + seg.ns - taken <= kPoolSize &&
                        (seg.ns == 1 || busy != (1u << NS) - 1)) {
                        int slot = 0;
                        if (seg.ns > 1) {
                            slot = __builtin_ctz(~busy);
                            busy |= 1u << slot;
                            if (lane == 0) {
                                fold[slot].next = 0;
                                fold[slot].ns = seg.ns;
                                fold[slot].kind = seg.kind;
                                fold[slot].dest = seg.dest;
                            }
                        }
                        // some chunks of the first segment are taken without the pool
                        const int skip = first ? direct_chunks(seg) : 0;
                        if (step_mode && seg.tail && skip < seg.ns) {
                            store_tail(seg);
                            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                            __builtin_amdgcn_s_waitcnt(0);
                        }
                        if (lane >= skip && lane < seg.ns)
                            pool.desc[(pool_end + lane - skip) % kPoolSize] = chunk_of(seg, lane, slot);
                        pool_end += seg.ns - skip;
                        __hip_atomic_store(&pool.end, pool_end, __ATOMIC_RELEASE,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                        ++pend_i;
                        first = false;
                        last_tok = seg.n_tok;
                        progressed = true;
                    }
                }
            }
            if (exhausted && pend_i == pend_n && q0 < 0 && !closed &&
                pool_end + NW - taken <= kPoolSize) {
                // one "no work left" entry per streaming wave
                if (lane < NW) {
                    ChunkDesc none{};
                    pool.desc[(pool_end + lane) % kPoolSize] = none;
                }
                pool_end += NW;
                __hip_atomic_store(&pool.end, pool_end, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
                closed = true;
                progressed = true;
            }
            // ---- results
            // partial results stored in this pass that are merged inside this launch: counted in
            // after the pass, when their mailboxes have been handed back
            int n_arr = 0;
            // Bound by latency: one wave, and every LDS read followed by a use.  The values go through
            // registers; the mailbox with its header, and then the slot, are one round trip each; the code
            // is there once, not once per mailbox.  Against reads word by word in four copies: 4 chats
            // x 4 heads of 64 dims 11.5 -> 10.2 us, 1664 rows of 1069 tokens 147.4 -> 145.8, 1024 of 1088 98.3
            // -> 97.0 (the wave used to end 2.5 to 3.6 us after the last streaming wave).  A chunk whose turn
            // has not come is read in vain in every pass; to look at the two headers first and to load after
            // that costs the round trip it saves: r = 8, 128 dims, 768 rows of 2176 tokens 145.5 -> 145.6 us,
            // 160 of 500 to 2000 30.8 -> 31.0, 508 of them 64.7 -> 65.0.
#pragma unroll 1
            for (; full != 0; full &= full - 1) {
                const int v = __builtin_ctz(full);
                Mail &mb = mail[v * 2 + (int)((boxes >> v) & 1u)];
                const i32x4 hdr = *reinterpret_cast<const i32x4 *>(&mb.kind);
                RowRegs<D, R> g;
                g.load(mb.o, mb.lse, lane);
                // a result that leaves the workgroup, if this chunk completes one
                bool leaves = true;
                int rkind = __builtin_amdgcn_readfirstlane(hdr.x), rdest = __builtin_amdgcn_readfirstlane(hdr.y);
                if (rkind == kKindFold) {
                    const int slot = rdest;
                    Fold &fs = fold[slot];
                    const i32x4 sh = *reinterpret_cast<const i32x4 *>(&fs.next);
                    constexpr int K = RowRegs<D, R>::K;
                    f32x4 y[K];
                    float Mo[K], Wo[K];                     // of no meaning before the first chunk
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const int e = RowRegs<D, R>::elem(lane, k);
                        y[k] = *reinterpret_cast<const f32x4 *>(&fs.acc[0][0] + e);
                        Mo[k] = fs.M[e / D];
                        Wo[k] = fs.W[e / D];
                    }
                    const int cs = __builtin_amdgcn_readfirstlane(hdr.z);
                    if (cs != __builtin_amdgcn_readfirstlane(sh.x)) continue;      // not its turn yet
                    leaves = cs + 1 == __builtin_amdgcn_readfirstlane(sh.y);
                    // chunk cs into the slot; a lane owns the same elements every time
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        float Mn = g.lse[k], Wn = 1.f;
                        if (cs > 0) {
                            const FoldCoef f = fold_coef(Mo[k], g.lse[k]);
                            Mn = f.Mn;
                            Wn = fold_weight(Wo[k], f);
                            g.x[k] = f32x4{fold_elem(y[k].x, g.x[k].x, f), fold_elem(y[k].y, g.x[k].y, f),
                                           fold_elem(y[k].z, g.x[k].z, f), fold_elem(y[k].w, g.x[k].w, f)};
                        }
                        if (leaves) {
                            const float inv = __builtin_amdgcn_rcpf(Wn);
                            g.x[k] = f32x4{g.x[k].x * inv, g.x[k].y * inv, g.x[k].z * inv, g.x[k].w * inv};
                            g.lse[k] = Mn + fast_log2(Wn);
                        } else if (RowRegs<D, R>::stored(lane)) {
                            const int e = lane * 4 + k * 256;
                            *reinterpret_cast<f32x4 *>(&fs.acc[0][0] + e) = g.x[k];
                            if (e % D == 0) {
                                fs.M[e / D] = Mn;
                                fs.W[e / D] = Wn;
                            }
                        }
                    }
                    if (leaves) {
                        busy &= ~(1u << slot);
                        rkind = __builtin_amdgcn_readfirstlane(sh.z);
                        rdest = __builtin_amdgcn_readfirstlane(sh.w);
                    } else if (lane == 0) {
                        fs.next = cs + 1;
                    }
                    wave_lds_fence();
                }
                if (leaves && MERGE && rkind == kKindPartial && merging) {
                    store_partial_coherent<D, R>(g, rdest, p, lane, spread);
                    if (lane == 0) {
                        arrivals.dest[n_arr] = rdest;
                        arrivals.parts[n_arr] = hdr.w;
                        arrivals.out_row[n_arr] = mb.out_row;
                        arrivals.len[n_arr] = mb.len;
                    }
                    ++n_arr;
                } else if (leaves) {
                    store_result<D, R>(g, rkind, rdest, p, lane);
                }
                mail_store(&mb.flag, kMailEmpty);
                boxes ^= 1u << v;
                progressed = true;
            }
            if (MERGE && n_arr > 0) {
                wave_lds_fence();           // lane 0's entries are read by all lanes
                count_in_and_combine<D, R, NW>(p, arrivals, n_arr, spread, batch * n_sel, lane);
            }
            if (progressed) {
                idle = 0;
            } else {
                ++idle;
                __builtin_amdgcn_s_sleep(kPollSleep);
            }
        }
        if (!counted_out) count_out();        // (only after a wait that gave up)
        if (lane == 0) {
            if (done_mask != (1 << NW) - 1) report_error(p.control, kErrWriterWait);
            if (draws ? gone_before == gridDim.x - 1 : blockIdx.x == 0)
                record_way(p.control, spread ? kModeSpread : split_mode ? kModeSplit : kModeSegments,
                           spread ? kWayChunks : split_mode ? kWaySplit : kWaySegments);
            if (draws && gone_before == gridDim.x - 1) {
                __hip_atomic_store(p.control + kCtlTickets, 0u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(p.control + kCtlGone, 0u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        return;
    }

    // ---------------------------------------------------------------- streaming waves
    // (no padding bytes anywhere: a struct with holes is copied through scratch memory, and a
    // scratch store in a streaming wave is a global store like any other)
    struct Slot {
        int64_t head_off;
        ItemHdr h;
        int ids;            // lane i: physical block of the chunk's i-th tile
        int exists, pad;
    };
    static_assert(sizeof(ItemHdr) == 11 * sizeof(int) && sizeof(Slot) == 8 + sizeof(ItemHdr) + 12,
                  "Slot has no padding");
    // chunk descriptor -> the wave's (uniform) bookkeeping, and the load of its block ids
    auto fill = [&](const ChunkDesc &d, Slot &s) {
        const int n_ids = __builtin_amdgcn_readfirstlane(d.n_ids);
        const int n_tok = __builtin_amdgcn_readfirstlane(d.n_tok);
        s.h.b = __builtin_amdgcn_readfirstlane(d.b);
        s.h.g = __builtin_amdgcn_readfirstlane(d.g);
        s.h.seq = __builtin_amdgcn_readfirstlane(d.seq);
        s.h.t0 = __builtin_amdgcn_readfirstlane(d.t0);
        s.h.kind = __builtin_amdgcn_readfirstlane(d.kind);
        s.h.dest = __builtin_amdgcn_readfirstlane(d.dest);
        s.h.cs = __builtin_amdgcn_readfirstlane(d.cs);
        s.h.nseg = __builtin_amdgcn_readfirstlane(d.nseg);
        s.h.out_row = __builtin_amdgcn_readfirstlane(d.out_row);
        s.h.len = __builtin_amdgcn_readfirstlane(d.len);
        s.exists = n_ids > 0 ? 1 : 0;
        s.h.n_tok = s.exists ? n_tok : 0;
        s.head_off = PAIRS ? 0 : (int64_t)s.h.g * p.stride_head;   // pairs: single-head tiles
        const int32_t *bt =
            p.block_table + (int64_t)s.h.b * p.max_blocks_per_seq + s.h.t0 / kBlockTokens;
        s.pad = 0;
        s.ids = bt[min(lane, max(n_ids, 1) - 1)];
    };
    auto q_rows = [&](const Slot &s) {
        return p.q + ((int64_t)s.h.seq * p.n_q_heads + s.h.g * R) * D;
    };
    auto issue = [&](Tile &t, int ids, int idx, int64_t head_off, int n_tok) {     // tile idx of a chunk of n_tok tokens
        const int blk = __builtin_amdgcn_readlane(ids, idx & 63);
        const int64_t base = (int64_t)blk * p.stride_block + head_off;
        const int nbytes = min(kBlockTokens, max(0, n_tok - idx * kBlockTokens)) * kRowBytes;
        Policy::issue(t, tile_rsrc(p.k_cache + base, nbytes), tile_rsrc(p.v_cache + base, nbytes), lane);
    };
    // bounded wait for a mailbox of this wave to be empty
    auto wait_empty = [&](Mail &mb) {
#pragma unroll 1
        for (int spin = 0; spin < kSpinLimit; ++spin) {
            if (__builtin_amdgcn_readfirstlane(mail_load(&mb.flag)) == kMailEmpty) return;
            __builtin_amdgcn_s_sleep(kPollSleep);
        }
        if (lane == 0) report_error(p.control, kErrMailboxWait);
    };
    // next chunk from the workgroup's pool (no ids: none left)
    auto take_chunk = [&]() {
        int i = 0;
        if (lane == 0)
            i = __hip_atomic_fetch_add(&pool.next, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        i = __builtin_amdgcn_readfirstlane(i);
#pragma unroll 1
        for (int spin = 0; spin < kSpinLimit; ++spin) {
            const int end = __builtin_amdgcn_readfirstlane(
                __hip_atomic_load(&pool.end, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
            if (end > i) return pool.desc[i % kPoolSize];
            __builtin_amdgcn_s_sleep(kPollSleep);
        }
        if (lane == 0) report_error(p.control, kErrTicketWait);
        ChunkDesc none{};
        return none;
    };

    // The lane's number for the wave's last chunk, which it stores itself: addresses that follow from it would be worked
    // out ahead of the streaming loop and kept, in 16 of the registers that the tiles of the MFMA path need.  (For
    // the hand-over of the others as well: the step of 145 pairs, r = 8, 40.1 us instead of 40.0, 8 rows of 500 to
    // 1500 15.6 instead of 15.3.)
    auto lane_again = [&]() {
        int l = lane;
        if constexpr (R >= 4) asm volatile("" : "+v"(l));
        return l;
    };
    unsigned char *my_staging = staging + (size_t)wave * Policy::kWaveLdsBytes;
    Mail *my_mail = mail + wave * 2;

    // SPLIT: split_mode
    auto stream = [&](auto ring_of, auto split) {
        constexpr int RING = decltype(ring_of)::value;   // tile pairs a wave keeps in flight, at most
        constexpr bool SPLIT = decltype(split)::value;
        Slot cur, nxt;
        typename Policy::Query q;
        typename Policy::QueryPrefetch q_pre;
        Tile ring[RING];
        {
            // first chunk: of the work the workgroup has without a ticket, else from the pool
            ChunkDesc d{};
            bool direct = false;
            if (spread) {
                const int mine = wave * (int)gridDim.x + (int)blockIdx.x;
                if (mine < total) {
                    const Segment s0 = quick_spread(mine);
                    if (step_mode && s0.tail) store_own_tail(s0);
                    d = chunk_of(s0, 0, 0);
                    direct = true;
                }
            } else if (SPLIT) {
                const long long mine = (long long)blockIdx.x * NW + wave;
                if (mine < total) {
                    d = chunk_of(decode((int)mine), 0, 0);
                    direct = true;
                }
            } else if (have_first) {
                const Segment s0 = decode(blockIdx.x);
                if (wave < direct_chunks(s0)) {
                    if (MERGE && step_mode && s0.tail && wave == s0.ns - 1) store_own_tail(s0);
                    d = chunk_of(s0, wave, 0);
                    direct = true;
                }
            }
            if (!direct) d = take_chunk();
            fill(d, cur);
        }
        if (!cur.exists) {
            mail_store(&my_mail[0].flag, kMailDone);
            return;
        }
        nxt = cur;
        Policy::q_prefetch(q_pre, q_rows(cur), lane);
#pragma unroll
        for (int s = 0; s < RING; ++s) issue(ring[s], cur.ids, s, cur.head_off, cur.h.n_tok);
        int n = 0;
        for (;; ++n) {
            Policy::q_commit(q, q_pre, my_staging, lane);   // this chunk's query operand

            // pieces of a chunk: sums of their own, folded in order (split calls: one piece)
            constexpr int PT = SPLIT ? 1 << 20 : decode_piece_tokens(R) / kBlockTokens;      // tiles
            // a piece is whole turns of the ring and folded behind the last one's refills, or (MFMA path, 128
            // dims) it ends anywhere in a turn and is folded behind its last tile
            constexpr bool kAnywhere = !SPLIT && PT % RING != 0;
            typename Policy::State st, tot;
            Policy::reset(st);
            Policy::reset(tot);
            auto next_piece = [&](int n_tiles) {            // after so many tiles of the chunk
                if (SPLIT || n_tiles % PT != 0) return;
                Policy::fold(tot, st);
                Policy::reset(st);
            };
            const int n_tok = cur.h.n_tok, n_my = (n_tok + kBlockTokens - 1) / kBlockTokens;
            const int lim = RING * max(1, (n_my + RING - 1) / RING);   // tiles, as whole ring turns
            // The scheduling fences keep "consume a slot, refill it at once" in program order;
            // without them the compiler batches the tiles' arithmetic ahead of the refills and
            // the wave ends up waiting with nothing in flight.  Where a turn is a whole piece (64 dims,
            // deep ring) the sums begin and end in it, and the compiler moves all of the turn's arithmetic
            // behind its last refill, so that the first refill waits for the whole ring: 480 rows of 1000 to
            // 1300 tokens, r = 2, 38.0 us, with the sums settled tile by tile 36.7; 400 of 300 to 1600, r = 1,
            // 29.0 and 28.1.  In launches of no more rows than workgroups, which wait for the way to memory
            // and not for its width, r = 1 is better off with one wait a turn (20 rows of 10k to 32k 31.0
            // and 32.7; r = 2, 24 of 6k to 9k 18.8 and 18.7).
            constexpr bool kSettle = PT == RING && (R == 2 || !TEAM);
            auto steady_turn = [&](int i) {                 // whole tiles; refills stay in this chunk
#pragma unroll
                for (int s = 0; s < RING; ++s) {
                    Policy::template update<kFullTile>(st, ring[s], q, p.scale_log2, lane, kBlockTokens);
                    if constexpr (kSettle) Policy::settle(st);
                    if (kAnywhere) next_piece(i + s + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    issue(ring[s], cur.ids, i + RING + s, cur.head_off, n_tok);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            // The next chunk is taken as late as its block ids allow (three ring turns before
            // the end of this one), so that little undone work is held back when the work runs
            // out.
            int i = 0;
            for (; i + 4 * RING < lim; i += RING) {
                steady_turn(i);
                if (!kAnywhere) next_piece(i + RING);
            }
            if (SPLIT && n == 0) {
                // the wave's second segment is its own as well
                const long long mine = (long long)(gridDim.x + blockIdx.x) * NW + wave;
                if (mine < total) {
                    fill(chunk_of(decode((int)mine), 0, 0), nxt);
                } else {
                    ChunkDesc none{};
                    fill(none, nxt);
                }
            } else {
                fill(take_chunk(), nxt);
            }
            Policy::q_prefetch(q_pre, q_rows(nxt), lane);   // next chunk's query rows
            for (; i + RING < lim; i += RING) {
                steady_turn(i);
                if (!kAnywhere) next_piece(i + RING);
            }
            // last turn of this chunk (the only place a ragged block can be): its refills are the
            // first tiles of the next chunk
#pragma unroll
            for (int s = 0; s < RING; ++s) {
                if (i + s < n_my) {
                    Policy::template update<kMaybeRagged>(st, ring[s], q, p.scale_log2, lane,
                                                  n_tok - (i + s) * kBlockTokens);
                    if (kAnywhere && i + s + 1 < n_my) next_piece(i + s + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
                issue(ring[s], nxt.ids, s, nxt.head_off, nxt.h.n_tok);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!SPLIT) Policy::fold(tot, st);
            typename Policy::State &sum = SPLIT ? st : tot;

            Mail &mb = my_mail[n & 1];
            wait_empty(mb);
            if (MERGE && !nxt.exists && cur.h.kind != kKindFold) {
                // The wave's last chunk, and a result of its own: no load is in flight that a store
                // could hold up, so the wave stores, counts and combines it itself instead of
                // queueing behind the other waves' results at the writer.
                const int lane_now = lane_again();
                if (cur.h.kind != kKindZero) Policy::finish(sum, mb.o, mb.lse, lane_now);
                wave_lds_fence();
                RowRegs<D, R> g;
                g.load(mb.o, mb.lse, lane_now);
                if (cur.h.kind == kKindPartial && merging) {
                    store_partial_coherent<D, R>(g, cur.h.dest, p, lane_now, spread);
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __builtin_amdgcn_s_waitcnt(0);      // every store of this wave has completed
                    unsigned old = 0;
                    if (lane == 0)
                        old = __hip_atomic_fetch_add(
                            p.arrivals + arrival_counter<R>(p, cur.h.dest, spread, batch * n_sel), 1u,
                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    mail_store(&mb.flag, kMailDone);
                    combine_if_last<D, R>(p, __builtin_amdgcn_readfirstlane((int)old), 1, cur.h.dest, cur.h.nseg,
                                          cur.h.out_row, cur.h.len, spread, batch * n_sel, lane);
                } else {
                    store_result<D, R>(g, cur.h.kind, cur.h.dest, p, lane_now);
                    mail_store(&mb.flag, kMailDone);
                }
                return;
            }
            // hand the finished chunk to the writer
            if (cur.h.kind != kKindZero) Policy::finish(sum, mb.o, mb.lse, lane);
            if (lane == 0) {
                mb.kind = cur.h.kind;
                mb.dest = cur.h.dest;
                mb.cs = cur.h.cs;
                mb.nseg = cur.h.nseg;
                mb.out_row = cur.h.out_row;
                mb.len = cur.h.len;
            }
            mail_store(&mb.flag, kMailFull);
            if (!nxt.exists) break;
            cur = nxt;
        }
        Mail &last = my_mail[(n + 1) & 1];
        wait_empty(last);
        mail_store(&last.flag, kMailDone);
    };
    if constexpr (CAN_SPLIT) {
        if (split_mode) {
            stream(IntTag<Policy::ring_split>{}, IntTag<1>{});
            return;
        }
    }
    if constexpr (Policy::ring(true) != Policy::ring(false)) {
        bool deep = quick;                // a few rows, in registers: nothing to look up
        if (!deep) {
            const int sample = lens[(lane * batch) >> 6];
            const int n_short = __builtin_popcountll(__builtin_amdgcn_ballot_w64(short_row<Policy>(sample)));
            deep = deep_ring<Policy>(batch * n_sel, n_short);
        }
        if (__builtin_expect(!deep, !MERGE)) {
            stream(IntTag<Policy::ring(false)>{}, IntTag<0>{});
            return;
        }
    }
    stream(IntTag<Policy::ring(true)>{}, IntTag<0>{});
}

}  // namespace hetis
