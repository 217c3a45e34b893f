"""Launches of short rows, a wave a row: the same rows behind a wider block table go through the
persistent kernel; both give the same bits, and the checker's results."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_08309_amd as H
from paper_2509_08309_amd import workloads as W

from gpu_harness import TOL, WAVE_ROWS, Dev, bits, check_rows, no_expired_wait, selected_rows, way

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def same(a, b):
    return torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("r,D", [(1, 64), (1, 128), (2, 64), (2, 128), (4, 64), (4, 128), (8, 64), (8, 128)])
@pytest.mark.parametrize("rows,limit", [(3, 64), (256, 64), (257, 256), (511, 512), (512, 384), (1024, 512),
                                        (2050, 384)])
def test_a_wave_a_row(r, D, rows, limit):
    """Rows that end at and around tiles, pieces, chunks and the longest row of such a launch, and empty ones."""
    ends = [0, 1, 15, 16, 17, 31, 33, 63, 64, 65, 127, 128, 129, 192, 255, 256, 257, 300, 383, 384, 385, 448, 511, 512]
    limit = 128 if limit == 64 and r >= 4 else 256 if rows == 511 and r < 4 else limit       # (row_a_wave)
    ends = [e for e in ends if e <= limit]
    heads = 2 if rows % 2 == 0 else 1
    lens = [ends[(5 * i + i // len(ends)) % len(ends)] for i in range(rows // heads)]
    sel = list(range(heads))[::-1]
    kw = dict(seed=rows + r, device=DEV)
    narrow = W.make_custom(lens, r * heads, heads, D, sel, max_seq_len=limit, **kw)
    wide = W.make_custom(lens, r * heads, heads, D, sel, max_seq_len=4096, **kw)
    assert narrow.block_table.shape[1] == limit // 16 and wide.block_table.shape[1] == 256
    a, b = Dev(narrow), Dev(wide)
    ws = a.workspace(heads)
    out = a.decode_ws(sel, ws)
    no_expired_wait(ws)
    assert way(ws) == WAVE_ROWS
    assert ws[:12].view(torch.int32).tolist() == [0, 0, 0]             # nothing counted
    wide_ws = b.workspace(heads)
    assert np.array_equal(bits(out), bits(b.decode_ws(sel, wide_ws)))
    assert way(wide_ws) not in (0, WAVE_ROWS)
    ref = oracle.attn_decode(narrow.q.cpu().numpy(), narrow.k_cache.cpu().numpy(), narrow.v_cache.cpu().numpy(),
                             narrow.block_table, narrow.seq_lens, np.asarray(sel, dtype=np.int32), narrow.spec.scale)
    check_rows(out, ref, selected_rows(narrow.spec, sel), TOL, "a wave a row")
    # the decode step, and one head's rows as pairs in another order, against append + decode
    kn, vn = W.new_token_rows(narrow)
    hid, n = b.heads(sel)
    H.check(H.hetis_kv_append(b.shape, kn, vn, b.bt, b.sl, hid, n, wide.num_blocks, b.k, b.v), "append")
    want = b.decode(sel)
    got = a.new_out()
    H.check(H.hetis_attn_decode_step(a.shape, a.q, kn, vn, a.k, a.v, a.bt, a.sl, hid, n, a.scale, got), "step")
    assert same(a.k, b.k) and same(a.v, b.v) and same(got, want)
    if heads == 1:
        order = torch.randperm(rows, generator=torch.Generator().manual_seed(1)).int()
        ps, ph = order.to(DEV), torch.zeros(rows, dtype=torch.int32, device=DEV)
        got = a.new_out()
        H.check(H.hetis_attn_decode_pairs(a.shape, a.q, a.k.view(-1, 16, D), a.v.view(-1, 16, D),
                                          a.bt[order.long().to(DEV)].contiguous(), a.sl, ps, ph, rows, a.scale, got), "pairs")
        torch.cuda.synchronize()
        assert same(got, want)
    no_expired_wait()


def test_replayed_from_a_graph():
    """One kernel and nothing else: a graph replays it with new queries, eager calls in between."""
    lens = [1 + 37 * i % 256 for i in range(300)]
    d = Dev(W.make_custom(lens, 2, 2, 128, [0, 1], seed=5, device=DEV, max_seq_len=256))
    ws = d.workspace(2)
    out = d.decode_ws([0, 1], ws).clone()
    hid, n = d.heads([0, 1])
    replayed = d.new_out()
    call = lambda o, st: H.hetis_attn_decode_ws(d.shape, d.q, d.k, d.v, d.bt, d.sl, hid, n, d.scale, o, ws, ws.numel(), st)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        H.check(call(replayed, torch.cuda.current_stream().cuda_stream), "capture")
    for i in range(4):
        g.replay()
        torch.cuda.synchronize()
        assert same(replayed, out)
        d.q.copy_(d.q.roll(1, 0))
        out = d.decode_ws([0, 1], ws).clone()
    no_expired_wait(ws)
    assert way(ws) == WAVE_ROWS
