"""Launches of fewer than 512 rows (sequences x selected heads, or pairs) decide on the device how
they are handed out: single chunks, one row a workgroup, or whole segments like every other launch.
At the edges of that decision the results are those of the whole-segment launch, bit for bit: the
same call with a workspace that holds the control words only."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_08309_amd as H
from paper_2509_08309_amd import workloads as W

from gpu_harness import SEGMENTS, TOL, WAVE_ROWS, Dev, bits, check_rows, no_expired_wait, selected_rows, way

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def lengths(kind, n, r, rng):
    turn = 4 * (512 if r >= 4 else 256)             # tokens a workgroup's waves hold in one turn
    if kind == "short":                             # at most one full chunk
        return rng.choice([0, 1, 16, 63, 64, 65, turn // 4 - 1, turn // 4], size=n)
    if kind == "turn":                              # at most one turn
        return rng.choice([0, 1, 63, 256, 257, turn // 4 + 1, turn - 1, turn], size=n)
    if kind == "one_long":                          # just beyond a chunk
        lens = rng.integers(0, 200, size=n)
        lens[rng.integers(n)] = turn // 4 + 1
        return lens
    return rng.choice([1, 255, 1025, 2048, 2049, 4095, 4096], size=n)


@pytest.mark.parametrize("Hq,Hkv,D", [(1, 1, 64), (2, 1, 128), (8, 1, 128)])
@pytest.mark.parametrize("kind", ["short", "turn", "one_long", "long"])
def test_ways_of_handing_out_agree(Hq, Hkv, D, kind):
    r = Hq // Hkv
    for n in (1, 63, 64, 65, 255, 256, 257, 511, 512):
        rng = np.random.default_rng(1000 + n)
        lens = [int(x) for x in lengths(kind, n, r, rng)]
        w = W.make_custom(lens, Hq, Hkv, D, [0], seed=n, device=DEV)
        d = Dev(w)
        out = d.decode([0])
        small = torch.empty(256, dtype=torch.uint8, device=DEV)
        H.check(H.hetis_attn_workspace_init(small, 256), "workspace_init")
        assert w.block_table.shape[1] <= 256        # one segment a row: nothing else in a workspace
        whole = d.decode_ws([0], small)
        assert np.array_equal(bits(out), bits(whole)), (kind, n)
        ws = d.workspace(1)
        for _ in range(2):                          # the second call finds what the first one left
            assert np.array_equal(bits(d.decode_ws([0], ws)), bits(whole)), (kind, n)
        torch.cuda.synchronize()
        mode = int(ws[:16].view(torch.int32)[3].item())
        turn = 4 * (512 if r >= 4 else 256)
        chunks = max(lens) > turn // 4 and n < 512 and (r < 4 or max(lens) <= turn or n < 256)
        if n == 511 and kind == ("long" if r < 4 else "turn"):
            chunks = False                          # nearly two full segments a workgroup
        assert mode == (3 if chunks else 1), (kind, n, mode)
        # the same rows as pairs, in another order
        perm = rng.permutation(n).astype(np.int32)
        pairs_out = torch.zeros_like(w.q)
        table = torch.from_numpy(np.ascontiguousarray(w.block_table[perm])).to(DEV)
        H.check(H.hetis_attn_decode_pairs(d.shape, d.q, d.k.view(-1, 16, D), d.v.view(-1, 16, D), table, d.sl,
                                          torch.from_numpy(perm).to(DEV), torch.zeros(n, dtype=torch.int32, device=DEV),
                                          n, d.scale, pairs_out), "pairs")
        torch.cuda.synchronize()
        no_expired_wait()
        assert np.array_equal(bits(pairs_out), bits(whole)), (kind, n)


@pytest.mark.parametrize("Hq,D", [(2, 128), (2, 64), (8, 128), (16, 64)])
def test_rows_of_many_segments(Hq, D):
    """Two long rows a head: as many segments and chunks a segment as the batched loads of the
    combination take, and one more."""
    Hkv = 2
    lens = [16 * 4096 + 1, 17 * 4096 + 300, 4097]
    w = W.make_custom(lens, Hq, Hkv, D, [1, 0], seed=77, device=DEV)
    out = Dev(w).decode([1, 0])
    ref = oracle.attn_decode(w.q.cpu().numpy(), w.k_cache.cpu().numpy(), w.v_cache.cpu().numpy(),
                             w.block_table, w.seq_lens, np.asarray([1, 0], dtype=np.int32), w.spec.scale)
    check_rows(out, ref, selected_rows(w.spec, [1, 0]), TOL, "long rows")
    no_expired_wait()


@pytest.mark.parametrize("Hq,D,rows,length,mode", [
    (1, 64, 128, 600, 3), (1, 64, 204, 600, 3), (1, 64, 205, 600, 1), (1, 64, 256, 600, 1), (1, 64, 257, 600, 3),
    (1, 128, 179, 4096, 3), (1, 128, 180, 4096, 1), (1, 128, 415, 2000, 3), (1, 128, 416, 2000, 1),
    (1, 64, 511, 300, 3), (1, 64, 511, 600, 3), (1, 128, 426, 700, 3), (1, 128, 427, 700, 1),
    (2, 128, 383, 2000, 3), (2, 128, 384, 2000, 1), (2, 64, 415, 2000, 3), (2, 64, 416, 2000, 1), (2, 64, 511, 300, 3),
    (8, 128, 179, 2048, 3), (8, 128, 180, 2048, 1), (4, 64, 88, 600, 3), (4, 64, 89, 600, 1),
    (8, 128, 257, 1200, 3), (8, 128, 415, 1200, 3), (8, 128, 416, 1200, 1), (8, 128, 257, 2049, 1),
])
def test_rows_whole_or_in_chunks(Hq, D, rows, length, mode):
    """Both sides of the lines between single chunks (mode 3) and whole rows (mode 1), rows of one
    length: the same bits as a launch that can only hand out whole rows."""
    w = W.make_custom([length] * rows, Hq, 1, D, [0], seed=rows, device=DEV)
    d, ws = Dev(w), torch.empty(256, dtype=torch.uint8, device=DEV)
    H.check(H.hetis_attn_workspace_init(ws, 256), "workspace_init")
    whole = d.decode_ws([0], ws)
    ws = d.workspace(1)
    assert np.array_equal(bits(d.decode_ws([0], ws)), bits(whole))
    assert int(ws[:16].view(torch.int32)[3].item()) == mode


@pytest.mark.parametrize("r,D,rows,lo,hi,mode,chunks,tokens", [       # (tokens a row of the block table holds, or as needed)
    (1, 64, 60, 0, 256, 1, None, None),          # a row a workgroup
    (8, 128, 300, 0, 512, 1, None, None),        # a wave a row;
    (8, 128, 300, 0, 512, 1, None, 1024),        # behind a wider block table whole rows through the tables
    (1, 128, 511, 1400, 1700, 1, None, None),    # whole rows of several chunks
    (8, 64, 280, 0, 600, 3, 1024, None),         # single chunks: up to one a wave,
    (2, 64, 300, 200, 700, 3, 2048, None),       # two a wave: the second through the pool,
    (8, 128, 300, 1900, 2048, 3, 2048, None),
    (1, 128, 410, 1900, 2000, 3, 4096, None),    # more: the rest by tickets
    (2, 64, 380, 1900, 2000, 3, 4096, None),
    (1, 64, 40, 19000, 24000, 3, 4096, None),    # the same, rows of several segments
])
@pytest.mark.parametrize("pairs", [False, True])
def test_steps_of_few_rows(r, D, rows, lo, hi, mode, chunks, tokens, pairs):
    """The new rows are stored by whichever wave gets the chunk that reads them: at its first chunk,
    from the workgroup's pool, or with a ticket.  Cache and outputs are those of the store and the
    Attention in two calls."""
    rng = np.random.default_rng(rows)
    lens = rng.integers(lo, hi + 1, size=rows)
    lens[rng.integers(rows)] = hi
    if chunks:                                              # the case is the one that it says it is
        ct = 512 if r >= 4 else 256
        fine = lambda n: ct // (4 if n <= 256 else 2 if n <= 1024 else 1)
        n = sum(L // 4096 * (4096 // ct) + -(-(L % 4096) // fine(L % 4096)) if L else 1 for L in lens.tolist())
        assert chunks // 2 < n <= chunks
    w = W.make_custom(lens, 2 * r, 2, D, [1], seed=rows, device=DEV, max_seq_len=tokens)
    kn, vn = W.new_token_rows(w)
    two, one = Dev(w), Dev(w)
    two.k, two.v = w.k_cache.clone(), w.v_cache.clone()
    hid, _ = two.heads([1])
    H.check(H.hetis_kv_append(two.shape, kn, vn, two.bt, two.sl, hid, 1, w.num_blocks, two.k, two.v), "append")
    want = two.decode([1])
    out, ws = one.new_out(), one.workspace(1)
    if pairs:
        ps, ph = torch.arange(rows, device=DEV).int(), torch.ones(rows, dtype=torch.int32, device=DEV)
        table = 2 * one.bt + 1
        k_tiles, v_tiles = one.k.view(-1, 16, D), one.v.view(-1, 16, D)
        H.check(H.hetis_attn_decode_pairs_step_ws(one.shape, one.q, kn, vn, k_tiles, v_tiles, table, one.sl, ps, ph,
                                                  rows, one.scale, out, ws, ws.numel()), "step")
    else:
        H.check(H.hetis_attn_decode_step_ws(one.shape, one.q, kn, vn, one.k, one.v, one.bt, one.sl, hid, 1, one.scale,
                                            out, ws, ws.numel()), "step")
    torch.cuda.synchronize()
    no_expired_wait(ws)
    assert int(ws[:16].view(torch.int32)[3].item()) == mode
    if rows > 256 and hi <= 512:
        assert way(ws) == (SEGMENTS if tokens else WAVE_ROWS)
    same = lambda a, b: torch.equal(a.view(torch.int16), b.view(torch.int16))
    assert same(one.k, two.k) and same(one.v, two.v) and same(out, want)


@pytest.mark.parametrize("Hq,Hkv,D", [(2, 2, 64), (2, 1, 128), (8, 2, 64), (16, 2, 128)])
def test_nobody_counts_where_nobody_draws(Hq, Hkv, D):
    """Launches whose work is handed out without tickets leave the counter of finished workgroups alone
    (here: whatever the caller had put there); the others leave it at zero."""
    rng = np.random.default_rng(Hq + D)
    sel = list(range(Hkv))
    for lens in ([33], [17, 100] * 60, [300, 1200, 40] * 12, [20000, 5000], [100, 90] * 64, [0] * 9):
        w = W.make_custom(lens, Hq, Hkv, D, sel, seed=len(lens), device=DEV)
        d = Dev(w)
        ref = d.decode(sel)
        sizes = [H.hetis_attn_decode_workspace_bytes(d.shape, Hkv)[1]]
        if w.block_table.shape[1] <= 256 and len(lens) * Hkv <= 256:
            sizes.append(256)                       # the control words only: one row a workgroup, by table
        for nbytes in sizes:
            ws = torch.full((nbytes,), 0xAB, dtype=torch.uint8, device=DEV)
            H.check(H.hetis_attn_workspace_init(ws, nbytes), "workspace_init")
            words = ws[:16].view(torch.int32)
            words[1] = 1000000
            out = d.decode_ws(sel, ws)
            assert np.array_equal(bits(out), bits(ref)), (lens[:3], nbytes)
            assert words[:3].tolist() == [0, 1000000, 0], (lens[:3], nbytes, words.tolist())
            assert int(words[3]) in (1, 3)
    lens = [int(x) for x in rng.integers(1, 400, size=1200)]
    w = W.make_custom(lens, Hq, Hkv, D, sel, seed=5, device=DEV, max_seq_len=1024)
    d = Dev(w)
    ws = d.workspace(Hkv)
    out = d.decode_ws(sel, ws)
    assert ws[:20].view(torch.int32).tolist() == [0, 0, 0, 1, SEGMENTS]
    assert np.array_equal(bits(out), bits(d.decode(sel)))


@pytest.mark.parametrize("Hq,D,n,lo,hi,chunks", [
    (2, 128, 480, 1, 290, True),        # short rows cut into quarter chunks: 1.2 of them a wave
    (2, 128, 480, 75, 300, True),
    (2, 128, 460, 275, 1100, False),    # 2.5 chunks a wave
    (2, 128, 400, 300, 1200, True)])    # 2.2
def test_chunks_a_wave(Hq, D, n, lo, hi, chunks):
    """More rows than workgroups, two query rows of 128 dims a head: single chunks up to 2.3 a wave."""
    lens = [lo + (hi - lo) * ((7 * i) % n) // (n - 1) for i in range(n)]
    w = W.make_custom(lens, Hq, 1, D, [0], seed=n, device=DEV)
    d = Dev(w)
    ws = d.workspace(1)
    out = d.decode_ws([0], ws)
    assert int(ws[:16].view(torch.int32)[3]) == (3 if chunks else 1)
    small = torch.empty(256, dtype=torch.uint8, device=DEV)
    H.check(H.hetis_attn_workspace_init(small, 256), "workspace_init")
    assert np.array_equal(bits(out), bits(d.decode_ws([0], small)))
