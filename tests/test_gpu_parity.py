"""Parity of the HIP path (through the C ABI) against the fp64 CPU checker.

Bars: max abs error <= 4e-3 on fp16 outputs; head-subset rows bit-identical to
the all-heads run; run-to-run determinism; rows of unselected heads untouched.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_08309_amd as H
from paper_2509_08309_amd import workloads as W

from gpu_harness import (SEGMENTS, SENTINEL, TOL, WAVE_ROWS, Dev, as_f64, bits, check_rows, host_copy, no_expired_wait,
                         partials_as_rows, rows_as_partials, selected_rows, unselected_rows, way)

pytestmark = pytest.mark.gpu

# fp32 partials are not rounded to fp16 on output.  Vector path (query groups of 1 or 2): all
# arithmetic is fp32, errors stay near 1e-5.  MFMA path (groups of 4 or 8): the softmax
# weights enter the second product as fp16 (relative rounding 2^-11 per weight), which shows up
# as a few 1e-4 on outputs of magnitude ~1.
def partial_tol(group_size):
    return 1e-4 if group_size < 4 else 1e-3


def oracle_of(w, head_ids=None, batch_idx=None):
    hid = w.head_ids if head_ids is None else np.asarray(head_ids, dtype=np.int32)
    q, bt, sl = w.q.numpy(), w.block_table, w.seq_lens
    if batch_idx is not None:
        q, bt, sl = q[batch_idx], bt[batch_idx], sl[batch_idx]
    return oracle.attn_decode(q, w.k_cache.numpy(), w.v_cache.numpy(), bt, sl, hid, w.spec.scale)


def check_against_oracle(out, ref, spec, head_ids, tol=TOL):
    """All selected rows of all sequences: written, finite, within tolerance."""
    return check_rows(out, ref, selected_rows(spec, head_ids), tol, spec.name)


def check_untouched(out, spec, head_ids):
    rows = unselected_rows(spec, head_ids)
    if rows:
        assert (bits(out)[:, rows] == SENTINEL).all(), "rows of unselected heads were written"


# ------------------------------------------------------------------ config 1
def test_c1_tiny_subset_parity_and_bit_identity():
    w = W.make_workload(W.SPECS["c1_tiny"])
    d = Dev(w)
    ref = oracle_of(w, list(range(8)))
    sub = d.decode([1, 3, 4, 6])
    full = d.decode(list(range(8)))
    check_against_oracle(sub, ref, w.spec, [1, 3, 4, 6])
    check_against_oracle(full, ref, w.spec, list(range(8)))
    check_untouched(sub, w.spec, [1, 3, 4, 6])
    assert np.array_equal(bits(sub)[:, [1, 3, 4, 6]], bits(full)[:, [1, 3, 4, 6]])
    again = d.decode([6, 4, 3, 1])                      # order of head_ids is irrelevant
    assert np.array_equal(bits(again), bits(sub))


# ------------------------------------------------------------------ edge cases
EDGE_LENS = [0, 1, 2, 15, 16, 17, 31, 33, 255, 256, 257, 300, 511, 512, 513, 1000]


@pytest.mark.parametrize("Hq,Hkv,D,hid", [
    (4, 4, 64, [0, 2, 3]),
    (4, 4, 128, [1, 3]),
    (8, 4, 128, [0, 3]),       # r = 2
    (8, 2, 64, [1]),           # r = 4
    (16, 2, 128, [0, 1]),      # r = 8
    (8, 1, 64, [0]),           # r = 8, D = 64
    (40, 40, 128, list(range(1, 37))),   # 576 rows: handed out in whole segments
    (80, 40, 64, list(range(2, 40))),    # the same with r = 2
])
def test_edge_lengths(Hq, Hkv, D, hid):
    w = W.make_custom(EDGE_LENS, Hq, Hkv, D, hid, seed=31, max_seq_len=1024)
    d = Dev(w)
    out = d.decode(hid)
    ref = oracle_of(w, hid)
    check_against_oracle(out, ref, w.spec, hid)
    check_untouched(out, w.spec, hid)
    rows = selected_rows(w.spec, hid)
    assert (bits(out)[0, rows] == 0).all()               # length 0 -> +0.0
    # length 1 returns that token's V row exactly
    blk = w.block_table[1, 0]
    r = Hq // Hkv
    for g in hid:
        for h in range(g * r, g * r + r):
            assert np.array_equal(bits(out)[1, h], w.v_cache.numpy()[blk, g, 0].view(np.uint16))
    full = d.decode(list(range(Hkv)))
    assert np.array_equal(bits(full)[:, rows], bits(out)[:, rows])
    assert np.array_equal(bits(d.decode(hid)), bits(out))   # deterministic


def test_constant_keys_give_mean_and_shift_invariance():
    w = W.make_custom([37, 300, 700], 2, 2, 128, [0, 1], seed=32, poison=False)
    w.k_cache[...] = 0.375
    d = Dev(w)
    out = as_f64(d.decode([0, 1]))
    v = w.v_cache.numpy().astype(np.float64)
    for b, L in enumerate(w.seq_lens):
        t = np.arange(L)
        mean = v[w.block_table[b][t // 16], :, t % 16].mean(axis=0)
        assert np.abs(out[b] - mean).max() <= TOL


def test_block_permutation_invariance_bitwise():
    w = W.make_custom([50, 333, 16, 600], 4, 4, 128, [0, 2], seed=33, max_seq_len=1024)
    a = Dev(w).decode([0, 2])
    rng = np.random.default_rng(5)
    perm = rng.permutation(w.num_blocks)
    k2 = torch.empty_like(w.k_cache)
    v2 = torch.empty_like(w.v_cache)
    k2[perm] = w.k_cache
    v2[perm] = w.v_cache
    w2 = W.Workload(w.spec, w.seq_lens,
                    np.where(w.block_table >= 0, perm[np.maximum(w.block_table, 0)], -1).astype(np.int32),
                    w.num_blocks, w.q, k2, v2, w.head_ids)
    b = Dev(w2).decode([0, 2])
    assert np.array_equal(bits(a), bits(b))


def test_head_major_pool_through_strides():
    w = W.make_custom([20, 45, 290], 3, 3, 64, [0, 2], seed=34, max_seq_len=512)
    ref = Dev(w).decode([0, 2])
    d = Dev(w)
    d.k = w.k_cache.permute(1, 0, 2, 3).contiguous().cuda()     # [Hkv, num_blocks, 16, D]
    d.v = w.v_cache.permute(1, 0, 2, 3).contiguous().cuda()
    d.shape.kv_stride_block = 16 * 64
    d.shape.kv_stride_head = w.num_blocks * 16 * 64
    assert np.array_equal(bits(d.decode([0, 2])), bits(ref))


# ------------------------------------------------------------------ split-KV and merge
@pytest.mark.parametrize("chunk", [16, 48, 512])
@pytest.mark.parametrize("Hq,Hkv,D", [(4, 4, 128), (8, 2, 64)])
def test_split_partials_and_merge(chunk, Hq, Hkv, D):
    lens = [0, 1, 16, 49, 700, 513, 512]
    hid = [1, 0]
    w = W.make_custom(lens, Hq, Hkv, D, hid, seed=35, max_seq_len=704)
    d = Dev(w)
    msl = 700
    C = H.hetis_attn_split_num_chunks(msl, chunk)
    o_p, lse_p = d.split(hid, chunk, msl)
    ro, rl = oracle.attn_partial(w.q.numpy(), w.k_cache.numpy(), w.v_cache.numpy(), w.block_table,
                                 w.seq_lens, hid, w.spec.scale, chunk, C)
    go, gl = partials_as_rows(o_p, lse_p)
    assert np.array_equal(np.isnan(gl), np.isnan(rl)), "written chunk set differs"
    assert np.array_equal(np.isnan(go), np.isnan(ro))
    m = ~np.isnan(rl)
    assert np.abs(gl[m] - rl[m]).max() <= 1e-4
    assert np.abs(go[~np.isnan(ro)] - ro[~np.isnan(ro)]).max() <= partial_tol(Hq // Hkv)
    out = d.merge(o_p, lse_p, hid, chunk, msl)
    ref = oracle_of(w, hid)
    check_against_oracle(out, ref, w.spec, hid)
    check_untouched(out, w.spec, hid)
    # split subset vs split full: bit-identical partials and outputs
    o_f, lse_f = d.split(list(range(Hkv)), chunk, msl)
    out_f = d.merge(o_f, lse_f, list(range(Hkv)), chunk, msl)
    rows = selected_rows(w.spec, hid)
    assert np.array_equal(bits(out_f)[:, rows], bits(out)[:, rows])


def test_merge_kernel_alone_on_checker_partials():
    lens = [0, 5, 100, 640]
    hid = [0, 1]
    w = W.make_custom(lens, 4, 2, 128, hid, seed=36, max_seq_len=640)
    chunk, msl = 64, 640
    C = 10
    ro, rl = oracle.attn_partial(w.q.numpy(), w.k_cache.numpy(), w.v_cache.numpy(), w.block_table,
                                 w.seq_lens, hid, w.spec.scale, chunk, C, fill=np.nan)
    ref = oracle.attn_merge(ro, rl, w.seq_lens, hid, 4, 2, chunk)
    d = Dev(w)
    o_np, lse_np = rows_as_partials(ro, rl, 2)
    o_p = torch.from_numpy(o_np).cuda()
    lse_p = torch.from_numpy(lse_np).cuda()
    out = d.merge(o_p, lse_p, hid, chunk, msl)
    check_against_oracle(out, ref, w.spec, hid)
    assert (bits(out)[0] == 0).all()


# ------------------------------------------------------------------ full-size configs, every row
def full_size_check(name, all_heads_vs_oracle=False):
    """The named workload at full size in the launch configuration the benchmark times: every
    selected row of every sequence against the checker (written, finite, within tolerance),
    unselected rows untouched, and the subset rows bit-identical to the all-heads run (whose
    remaining rows are compared with the checker too when `all_heads_vs_oracle`)."""
    spec = W.SPECS[name]
    w = W.make_workload(spec, device="cuda:0")
    d = Dev(w)
    heads = list(spec.head_ids)
    sub = d.decode(heads)
    wh = host_copy(w)
    everything = list(range(spec.n_kv_heads))
    ref = oracle_of(wh, everything if all_heads_vs_oracle else heads)
    check_against_oracle(sub, ref, spec, heads)
    check_untouched(sub, spec, heads)
    if len(heads) < spec.n_kv_heads:
        full = d.decode(everything)
        srows = selected_rows(spec, heads)
        assert np.array_equal(bits(full)[:, srows], bits(sub)[:, srows]), \
            f"{name}: subset is not bit-identical to the slice of the all-heads run"
        if all_heads_vs_oracle:
            check_against_oracle(full, ref, spec, everything)
    return d, wh, sub, ref


def test_c2_7b_all_heads():
    full_size_check("c2_7b_all")


def test_c2_7b_half_vs_all():
    full_size_check("c2_7b_half", all_heads_vs_oracle=True)


def test_c3_13b_subset():
    full_size_check("c3_13b_subset", all_heads_vs_oracle=True)


def test_c5_70b_gqa():
    full_size_check("c5_70b_gqa")


def test_c4_long_split_512_and_decode():
    spec = W.SPECS["c4_13b_long"]
    d, wh, out_dec, ref = full_size_check("c4_13b_long")
    hid = list(spec.head_ids)
    o_p, lse_p = d.split(hid, spec.chunk_tokens, spec.max_seq_len)
    out = d.merge(o_p, lse_p, hid, spec.chunk_tokens, spec.max_seq_len)
    check_against_oracle(out, ref, spec, hid)
    # every chunk a sequence has was written, none beyond it
    C = H.hetis_attn_split_num_chunks(spec.max_seq_len, spec.chunk_tokens)
    n_chunks = (wh.seq_lens.astype(np.int64) + spec.chunk_tokens - 1) // spec.chunk_tokens
    written = ~np.isnan(as_f64(lse_p))                      # [B, S, C, r]
    expect = np.arange(C)[None, :] < n_chunks[:, None]      # [B, C]
    assert np.array_equal(written, np.broadcast_to(expect[:, None, :, None], written.shape))
    # head subset through the split path: bit-identical to the slice of the all-heads split run
    sub_ids = [3, 17, 38]
    o_s, lse_s = d.split(sub_ids, spec.chunk_tokens, spec.max_seq_len)
    out_s = d.merge(o_s, lse_s, sub_ids, spec.chunk_tokens, spec.max_seq_len)
    assert np.array_equal(bits(out_s)[:, sub_ids], bits(out)[:, sub_ids])
    check_untouched(out_s, spec, sub_ids)


def test_split_of_very_many_chunks():
    """64 neighbouring rows of the enumeration hold over 2^21 chunks: the last rows' chunks start
    beyond what 21 bits count.  Every row's partial results are those of a call with the row alone.
    (The rows' tables name the same few blocks over and over, so that the cache stays small.)"""
    D, n_rows, n_blk, pool = 64, 65, 34500, 512
    lens = [n_blk * 16 - (b % 16) for b in range(n_rows)]
    assert 62 * (lens[15] // 16) > 1 << 21
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(55)
    k, v = (torch.randn((pool, 1, 16, D), generator=gen, device="cuda:0").half() for _ in range(2))
    q = torch.randn((n_rows, 1, D), generator=gen, device="cuda:0").half()
    bt = torch.randint(0, pool, (n_rows, n_blk), generator=gen, device="cuda:0").int()
    sl, hid = (torch.tensor(x, dtype=torch.int32, device="cuda:0") for x in (lens, [0]))
    partials = lambda n: (torch.full((n, 1, n_blk, 1, D), float("nan"), device="cuda:0"),
                          torch.full((n, 1, n_blk, 1), float("nan"), device="cuda:0"))
    o_all, lse_all = partials(n_rows)
    H.check(H.hetis_attn_decode_split(H.make_shape(n_rows, 1, 1, D, n_blk), q, k, v, bt, sl, hid, 1, D ** -0.5, 16,
                                      n_blk * 16, o_all, lse_all), "split")
    no_expired_wait()
    for b in range(n_rows):
        o, lse = partials(1)
        H.check(H.hetis_attn_decode_split(H.make_shape(1, 1, 1, D, n_blk), q[b:b + 1], k, v, bt[b:b + 1], sl[b:b + 1],
                                          hid, 1, D ** -0.5, 16, n_blk * 16, o, lse), "split of one row")
        assert torch.equal(o[0], o_all[b]) and torch.equal(lse[0], lse_all[b]), b
    no_expired_wait()


# ------------------------------------------------------------------ other entry points and paths
def test_validate_reports_bad_content():
    w = W.make_custom([20, 45], 4, 4, 64, [0, 1], seed=41, max_seq_len=64)
    d = Dev(w)
    hid, n = d.heads([0, 1])
    assert H.hetis_attn_validate(d.shape, d.bt, d.sl, hid, n, w.num_blocks) == 0
    bad_hid = torch.tensor([0, 4], dtype=torch.int32, device="cuda:0")          # head 4 of 4
    assert H.hetis_attn_validate(d.shape, d.bt, d.sl, bad_hid, 2, w.num_blocks) == H.binding.HETIS_ERR_BAD_CONTENT
    bad_len = torch.tensor([20, 65], dtype=torch.int32, device="cuda:0")        # beyond the table
    assert H.hetis_attn_validate(d.shape, d.bt, bad_len, hid, n, w.num_blocks) == H.binding.HETIS_ERR_BAD_CONTENT
    assert H.hetis_attn_validate(d.shape, d.bt, d.sl, hid, n, 2) == H.binding.HETIS_ERR_BAD_CONTENT  # block id >= 2


def test_profile_events_bracket_the_chunk_kernel():
    w = W.make_custom([300, 700, 64], 4, 4, 128, [0, 1, 2, 3], seed=42, max_seq_len=1024)
    d = Dev(w)
    ref = d.decode([0, 1, 2, 3])
    st = torch.cuda.current_stream()
    ev = []
    for _ in range(2):
        e = torch.cuda.Event(enable_timing=True)
        e.record(st)
        ev.append(e)
    torch.cuda.synchronize()
    assert H.hetis_attn_profile_events(ev[0].cuda_event, None) == H.binding.HETIS_ERR_NULL
    assert H.hetis_attn_profile_events(ev[0].cuda_event, ev[1].cuda_event) == 0
    out = d.decode([0, 1, 2, 3])
    assert H.hetis_attn_profile_events(None, None) == 0
    assert 0.0 < ev[0].elapsed_time(ev[1]) < 50.0          # milliseconds
    assert np.array_equal(bits(out), bits(ref))


@pytest.mark.parametrize("table,ways", [(1024, (SEGMENTS, SEGMENTS)), (304, (WAVE_ROWS, WAVE_ROWS))])
def test_batch_beyond_the_persistent_kernel_limit(table, ways):
    # more than 2048 sequences: several launches over slices of the sequences (behind a narrow block
    # table: one launch, a wave a sequence)
    rng = np.random.default_rng(43)
    lens = rng.integers(0, 300, size=4100).tolist()
    w = W.make_custom(lens, 2, 2, 64, [1], seed=43, max_seq_len=table)
    d = Dev(w)
    out = d.decode([1])
    for heads, expected in zip(([1], [0, 1]), ways):
        ws = d.workspace(len(heads))
        assert np.array_equal(bits(d.decode_ws(heads, ws))[:, 1], bits(out)[:, 1]) and way(ws) == expected
    ref = oracle_of(w, [1])
    check_against_oracle(out, ref, w.spec, [1])
    check_untouched(out, w.spec, [1])
    full = d.decode([0, 1])
    assert np.array_equal(bits(full)[:, 1], bits(out)[:, 1])


@pytest.mark.parametrize("table,expected", [(1024, SEGMENTS), (48, WAVE_ROWS)])
def test_many_short_sequences_and_repeat_calls(table, expected):
    # thousands of tiny items exercise the ticket pool; repeated calls must leave its counters
    # ready (identical bits every time).  Behind a narrow block table: a wave each, no counters
    rng = np.random.default_rng(44)
    lens = rng.integers(1, 40, size=1500).tolist()
    w = W.make_custom(lens, 4, 4, 128, [0, 2, 3], seed=44, max_seq_len=table)
    d = Dev(w)
    first = d.decode([0, 2, 3])
    ref = oracle_of(w, [0, 2, 3])
    check_against_oracle(first, ref, w.spec, [0, 2, 3])
    ws = d.workspace(3)
    for _ in range(5):
        assert np.array_equal(bits(d.decode([0, 2, 3])), bits(first))
        assert np.array_equal(bits(d.decode_ws([0, 2, 3], ws)), bits(first))
        assert ws[:12].view(torch.int32).tolist() == [0, 0, 0] and way(ws) == expected


# ------------------------------------------------------------------ graphs and streams

def test_graph_capture_and_replay():
    """hetis_attn_decode and hetis_kv_append captured into a HIP graph (after one eager call has
    allocated the library's workspace): every replay, with new queries and new rows in the same
    buffers and eager work in between, matches an eager call bit for bit."""
    w = W.make_custom([40, 300, 1500, 17, 700], 8, 8, 128, [1, 4, 6], seed=91, device="cuda:0")
    d = Dev(w)
    heads = [1, 4, 6]
    hid, n = d.heads(heads)
    kn, vn = W.new_token_rows(w)
    out = d.new_out()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        H.check(H.hetis_attn_decode(d.shape, d.q, d.k, d.v, d.bt, d.sl, hid, n, d.scale, out, side))
    side.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        H.check(H.hetis_kv_append(d.shape, kn, vn, d.bt, d.sl, hid, n, w.num_blocks, d.k, d.v, side))
        H.check(H.hetis_attn_decode(d.shape, d.q, d.k, d.v, d.bt, d.sl, hid, n, d.scale, out, side))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(92)
    for it in range(4):
        d.q.copy_(torch.randn(d.q.shape, generator=gen, device="cuda:0").half())
        kn.copy_(torch.randn(kn.shape, generator=gen, device="cuda:0").half())
        vn.copy_(torch.randn(vn.shape, generator=gen, device="cuda:0").half())
        out.view(torch.int16).fill_(np.int16(SENTINEL))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        got = out.clone()
        # eager reference on the same (already appended) cache
        ref = d.decode(heads)
        assert torch.equal(got.view(torch.int16), ref.view(torch.int16)), f"replay {it}"
        rows = selected_rows(w.spec, heads)
        last = (w.seq_lens - 1)
        b = 2
        assert torch.equal(d.k[w.block_table[b, last[b] // 16], 4, last[b] % 16], kn[b, 4])
        check_untouched(got, w.spec, heads)
        assert not np.isnan(as_f64(got)[:, rows]).any()


def test_two_streams_with_their_own_buffers():
    """Split-KV calls on two streams at once (each with its own partial buffers, control words
    and outputs) give what the same calls give one after the other."""
    w1 = W.make_custom([2000, 900, 3000, 64], 8, 8, 128, [0, 3, 5, 7], seed=93, device="cuda:0")
    w2 = W.make_custom([1200, 2500, 300], 16, 2, 128, [1, 0], seed=94, device="cuda:0")
    devs = [Dev(w1), Dev(w2)]
    heads = [[0, 3, 5, 7], [1, 0]]
    msl = [3000, 2500]
    serial = []
    for d, h, m in zip(devs, heads, msl):
        o_p, lse_p = d.split(h, 512, m)
        serial.append(d.merge(o_p, lse_p, h, 512, m))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    bufs = []
    for d, h, m in zip(devs, heads, msl):
        s = d.w.spec
        C = H.hetis_attn_split_num_chunks(m, 512)
        bufs.append((torch.empty((s.batch, len(h), C, s.group_size, s.head_dim), dtype=torch.float32,
                                 device="cuda:0"),
                     torch.empty((s.batch, len(h), C, s.group_size), dtype=torch.float32,
                                 device="cuda:0"), d.new_out(), d.heads(h),
                     torch.zeros(H.binding.HETIS_ATTN_CONTROL_BYTES, dtype=torch.uint8, device="cuda:0")))
    torch.cuda.synchronize()
    for rep in range(6):
        for d, h, m, st, (o_p, lse_p, out, (hid, n), ctl) in zip(devs, heads, msl, streams, bufs):
            H.check(H.hetis_attn_decode_split_ws(d.shape, d.q, d.k, d.v, d.bt, d.sl, hid, n, d.scale,
                                                 512, m, o_p, lse_p, ctl, st))
            H.check(H.hetis_attn_merge(d.shape, o_p, lse_p, d.sl, hid, n, 512, m, out, st))
    torch.cuda.synchronize()
    for (o_p, lse_p, out, _, ctl), ref in zip(bufs, serial):
        no_expired_wait(ctl)
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16))


# ------------------------------------------------------------------ mid-size shapes of every kernel variant

@pytest.mark.parametrize("Hq,Hkv,D,hid", [
    (16, 16, 64, [3, 9, 10, 15]),      # vector path, D = 64
    (32, 16, 128, [0, 5, 6, 14]),      # vector path, r = 2
    (32, 8, 128, [1, 6]),              # MFMA path, r = 4
    (64, 8, 64, [0, 3, 7]),            # MFMA path, r = 8, D = 64
])
def test_mid_size_ragged_batch(Hq, Hkv, D, hid):
    """96 sequences, lognormal lengths up to 4096 (several decode chunks of either size, a ragged
    tail everywhere), several thousand items: every selected row against the checker, subset
    rows bit-identical to the all-heads run."""
    rng = np.random.default_rng(95)
    lens = np.clip(np.rint(rng.lognormal(np.log(900), 0.9, size=96)), 1, 4096).astype(int)
    lens[:3] = [4096, 1, 769]
    w = W.make_custom(lens, Hq, Hkv, D, hid, seed=96, device="cuda:0")
    d = Dev(w)
    out = d.decode(hid)
    ref = oracle_of(host_copy(w), hid)
    rows = selected_rows(w.spec, hid)
    check_against_oracle(out, ref, w.spec, hid)
    check_untouched(out, w.spec, hid)
    full = d.decode(list(range(Hkv)))
    assert np.array_equal(bits(full)[:, rows], bits(out)[:, rows])


def test_split_with_the_largest_chunk():
    """chunk_tokens = 1024: a wave's block-id register is full (64 blocks)."""
    lens = [1024, 1025, 3000, 2048, 5]
    hid = [0, 2]
    w = W.make_custom(lens, 4, 4, 128, hid, seed=97, device="cuda:0")
    d = Dev(w)
    o_p, lse_p = d.split(hid, 1024, 3000)
    out = d.merge(o_p, lse_p, hid, 1024, 3000)
    ref = oracle.attn_decode(w.q.cpu().numpy(), w.k_cache.cpu().numpy(), w.v_cache.cpu().numpy(),
                             w.block_table, w.seq_lens, np.asarray(hid, dtype=np.int32), w.spec.scale)
    check_against_oracle(out, ref, w.spec, hid)
    C = H.hetis_attn_split_num_chunks(3000, 1024)
    lse = as_f64(lse_p)
    assert C == 3 and np.isnan(lse[0, :, 1:]).all() and not np.isnan(lse[1, :, :2]).any()


@pytest.mark.parametrize("table,expected", [(1024, SEGMENTS), (208, WAVE_ROWS)])
def test_batch_at_the_persistent_kernel_limit(table, expected):
    """Exactly 2048 sequences: the largest batch the persistent kernel's tables hold (behind a narrow
    block table: a wave a sequence)."""
    rng = np.random.default_rng(98)
    lens = rng.integers(1, 200, size=2048)
    hid = [1]
    w = W.make_custom(lens, 2, 2, 64, hid, seed=99, device="cuda:0", max_seq_len=table)
    d = Dev(w)
    ws = d.workspace(1)
    out = d.decode_ws(hid, ws)
    assert way(ws) == expected
    ref = oracle_of(host_copy(w), hid)
    check_against_oracle(out, ref, w.spec, hid)
    check_untouched(out, w.spec, hid)
