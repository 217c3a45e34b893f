"""hetis_attn_decode_step: the decode-step store of the new token's K/V rows folded into the
Attention call (Section 5.1: store, then attend to all stored keys and values, the new one
included).  The cache must end up bit for bit as hetis_kv_append / the checker's append leave
it, and the output as hetis_attn_decode computes it on the appended cache."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_08309_amd as H
from paper_2509_08309_amd import workloads as W

from gpu_harness import (SEGMENTS, SENTINEL, TEAM_ITEMS, TEAM_ROWS, TOL, WAVE_ROWS, Dev, bits, check_rows, no_expired_wait,
                         selected_rows, way)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def run_step(d, heads, kn, vn, ws=None):
    hid, n = d.heads(heads)
    out = d.new_out()
    if ws is None:
        H.check(H.hetis_attn_decode_step(d.shape, d.q, kn, vn, d.k, d.v, d.bt, d.sl, hid, n, d.scale,
                                         out), "hetis_attn_decode_step")
    else:
        H.check(H.hetis_attn_decode_step_ws(d.shape, d.q, kn, vn, d.k, d.v, d.bt, d.sl, hid, n,
                                            d.scale, out, ws, ws.numel()), "hetis_attn_decode_step_ws")
    torch.cuda.synchronize()
    no_expired_wait(ws)
    return out


def check_step(w, heads, use_ws=False, expected=None):
    spec = w.spec
    kn, vn = W.new_token_rows(w)
    ref_k, ref_v = oracle.kv_append(bits(w.k_cache), bits(w.v_cache), bits(kn), bits(vn),
                                    w.block_table, w.seq_lens, heads)
    ref = oracle.attn_decode(w.q.cpu().numpy(), ref_k.view(np.float16), ref_v.view(np.float16),
                             w.block_table, w.seq_lens, np.asarray(heads, dtype=np.int32), spec.scale)
    # the two-call form on a copy of the cache
    two = Dev(w)
    two.k, two.v = w.k_cache.clone(), w.v_cache.clone()
    hid, n = two.heads(heads)
    H.check(H.hetis_kv_append(two.shape, kn, vn, two.bt, two.sl, hid, n, w.num_blocks, two.k, two.v),
            "hetis_kv_append")
    out_two = two.decode(heads)
    # the one-call form, in place on the workload's own cache
    one = Dev(w)
    ws = one.workspace(len(heads)) if use_ws else None
    out_one = run_step(one, heads, kn, vn, ws)
    assert expected is None or way(ws) == expected
    same = lambda t, r: bool(torch.equal(t.view(torch.int16).reshape(-1),
                                         torch.from_numpy(r.view(np.int16)).to(DEV).reshape(-1)))
    assert same(one.k, ref_k) and same(one.v, ref_v), "cache differs from the checker's append"
    assert torch.equal(one.k.view(torch.int16), two.k.view(torch.int16))
    rows = selected_rows(spec, heads)
    check_rows(out_one, ref, rows, TOL, "decode_step")
    assert torch.equal(out_one.view(torch.int16), out_two.view(torch.int16)), \
        "one call differs from append + decode"
    rest = [h for h in range(spec.n_q_heads) if h not in set(rows)]
    if rest:
        assert (bits(out_one)[:, rest] == SENTINEL).all()
    return one, kn, vn, out_one


@pytest.mark.parametrize("Hq,Hkv,D,heads", [
    (4, 4, 64, [0, 2, 3]),
    (8, 8, 128, [1, 6]),
    (8, 4, 128, [0, 3]),       # r = 2
    (16, 2, 128, [1]),         # r = 8
    (8, 1, 64, [0]),           # r = 8, D = 64
    (32, 32, 128, list(range(32))),      # 576 rows: whole segments, the store inside the kernel
    (256, 32, 128, list(range(3, 32))),  # the same with r = 8
])
def test_step_edge_lengths(Hq, Hkv, D, heads):
    # lengths around block, chunk and segment boundaries; the new token is the last one counted
    lens = [0, 1, 2, 15, 16, 17, 33, 255, 256, 257, 511, 512, 513, 1000, 4095, 4096, 4097, 5000]
    w = W.make_custom(lens, Hq, Hkv, D, heads, seed=501, device=DEV)
    one, kn, vn, out = check_step(w, heads)
    # a second step on the same (already appended) cache gives the same bits
    again = run_step(one, heads, kn, vn)
    assert torch.equal(again.view(torch.int16), out.view(torch.int16))


@pytest.mark.parametrize("name", ["c1_tiny", "c3_13b_subset", "c5_70b_gqa"])
def test_step_full_size(name):
    spec = W.SPECS[name]
    w = W.make_workload(spec, device=DEV)
    check_step(w, list(spec.head_ids), use_ws=(name == "c3_13b_subset"))


@pytest.mark.parametrize("table,expected", [(1024, SEGMENTS), (304, WAVE_ROWS)])
def test_step_many_short_rows(table, expected):
    """Thousands of one-chunk rows: the new row is stored by the wave that publishes the chunk,
    also when chunks are published in batches and when a workgroup's first chunk is the one
    that holds the new token (behind a narrow block table: by the row's own wave)."""
    rng = np.random.default_rng(502)
    lens = rng.integers(1, 300, size=1200)
    w = W.make_custom(lens, 4, 4, 128, [0, 1, 3], seed=503, device=DEV, max_seq_len=table)
    check_step(w, [0, 1, 3], use_ws=True, expected=expected)


@pytest.mark.parametrize("Hq,Hkv,D,B,heads,max_seq_len,expected", [
    (4, 2, 64, 2 * 2048 + 4, [1], 1024, SEGMENTS),    # three slices of at most 2048 sequences
    (4, 2, 64, 2 * 2048 + 4, [1], 33, WAVE_ROWS),     # one launch, a wave a sequence
    (512, 512, 64, 514, list(range(512)), 4097, SEGMENTS),      # rows of two segments: 2^18 / 512 sequences a slice
])
def test_step_of_more_sequences_than_a_launch_holds(Hq, Hkv, D, B, heads, max_seq_len, expected):
    """The launches after the first store their own sequences' new rows."""
    rng = np.random.default_rng(504)
    lens = rng.integers(1, min(max_seq_len, 48 if Hkv == 2 else 8192 // Hkv) + 1, size=B)
    lens[[0, 5]] = 0
    w = W.make_custom(lens, Hq, Hkv, D, heads, seed=505, device=DEV, max_seq_len=max_seq_len)
    check_step(w, heads, use_ws=True, expected=expected)


@pytest.mark.parametrize("pairs", [False, True])
@pytest.mark.parametrize("B", [3, 300])                # x 2 heads: few rows, and whole segments
@pytest.mark.parametrize("mb,expected", [(2, (WAVE_ROWS, WAVE_ROWS)), (5, (TEAM_ROWS, WAVE_ROWS)),
                                         (40, (TEAM_ITEMS, SEGMENTS))])
def test_step_does_not_store_past_the_block_table(B, mb, expected, pairs):
    """A position past a row's mb table entries is not stored, as in hetis_kv_append, and whichever way the
    launch goes Attention reads the row's last entry once more for it, and nothing outside the table."""
    Hkv, D, full = 2, 64, 16 * mb
    gen = torch.Generator(device=DEV)
    gen.manual_seed(506)
    bt = torch.randperm(B * mb, generator=gen, device=DEV).int().view(B, mb)
    lens = torch.randint(full - 15, full + 1, (B,), generator=gen, device=DEV).int()
    lens[::7] = full + 1
    lens[-1] = full + 1                                # the table ends with this row
    q, kn, vn = (torch.randn((B, Hkv, D), generator=gen, device=DEV).half() for _ in range(3))
    k, v = (torch.randn((B * mb, Hkv, 16, D), generator=gen, device=DEV).half() for _ in range(2))
    shape, hid = H.make_shape(B, Hkv, Hkv, D, mb), torch.tensor([0, 1], dtype=torch.int32, device=DEV)
    ps = torch.arange(B, device=DEV).int().repeat_interleave(Hkv)
    ph = hid.repeat(B)
    # tiles of a pair are its sequence's: B * Hkv rows of mb entries, the pairs of the last row last
    pt = (bt[ps.long()] * Hkv + ph[:, None]).int().contiguous()
    k2, v2, out, out2 = k.clone(), v.clone(), torch.zeros_like(q), torch.zeros_like(q)
    H.check(H.hetis_kv_append(shape, kn, vn, bt, lens, hid, Hkv, B * mb, k2, v2), "append")
    rc, need = H.hetis_attn_decode_pairs_workspace_bytes(shape, B * Hkv) if pairs else \
        H.hetis_attn_decode_workspace_bytes(shape, Hkv)
    H.check(rc)
    ws = torch.zeros(need, dtype=torch.uint8, device=DEV)
    if pairs:
        H.check(H.hetis_attn_decode_pairs_step_ws(shape, q, kn, vn, k.view(-1, 16, D), v.view(-1, 16, D), pt, lens, ps,
                                                  ph, B * Hkv, D ** -0.5, out, ws, need), "pairs step")
    else:
        H.check(H.hetis_attn_decode_step_ws(shape, q, kn, vn, k, v, bt, lens, hid, Hkv, D ** -0.5, out, ws, need), "step")
    # the same rows behind a table that has the entry, twice
    longer = torch.cat([bt, bt[:, -1:]], 1).contiguous()
    H.check(H.hetis_attn_decode(H.make_shape(B, Hkv, Hkv, D, mb + 1), q, k2, v2, longer, lens, hid, Hkv, D ** -0.5, out2),
            "decode")
    torch.cuda.synchronize()
    no_expired_wait(ws)
    no_expired_wait()
    assert way(ws) == expected[B > 3]
    assert torch.equal(k, k2) and torch.equal(v, v2)
    assert torch.equal(out, out2)
