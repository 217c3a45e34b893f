"""Launches in which the waves of a workgroup share a chunk (one item a workgroup, or one row): at the edges of
pieces, windows and the number of workgroups the results are those of the launch that hands out whole
segments, bit for bit, and the checker's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_08309_amd as H
from paper_2509_08309_amd import workloads as W

from gpu_harness import (CHUNKS, TEAM_ITEMS, TEAM_ROWS, TOL, WAVE_ROWS, Dev, bits, check_rows, no_expired_wait,
                         selected_rows, way)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def compare(lens, Hq, D, expected):
    """A launch of few rows, handed out as `expected`, against whole segments (a workspace of the control words
    alone) and the checker; as a decode step against append + decode; as pairs."""
    w = W.make_custom([int(x) for x in lens], Hq, 1, D, [0], seed=len(lens) + Hq, device=DEV)
    d = Dev(w)
    ws = d.workspace(1)
    out = d.decode_ws([0], ws)
    no_expired_wait(ws)
    assert way(ws) == expected, (len(lens), max(lens))
    assert ws[:12].view(torch.int32).tolist() == [0, 0, 0]
    ref = oracle.attn_decode(w.q.cpu().numpy(), w.k_cache.cpu().numpy(), w.v_cache.cpu().numpy(),
                             w.block_table, w.seq_lens, np.asarray([0], dtype=np.int32), w.spec.scale)
    check_rows(out, ref, selected_rows(w.spec, [0]), TOL, "team")
    if w.block_table.shape[1] <= 256:                    # rows of one segment: nothing else in a workspace
        small = torch.empty(256, dtype=torch.uint8, device=DEV)
        H.check(H.hetis_attn_workspace_init(small, 256), "workspace_init")
        assert np.array_equal(bits(out), bits(d.decode_ws([0], small)))
    kn, vn = W.new_token_rows(w)
    two, one = Dev(w), Dev(w)
    two.k, two.v = w.k_cache.clone(), w.v_cache.clone()
    hid, _ = two.heads([0])
    H.check(H.hetis_kv_append(two.shape, kn, vn, two.bt, two.sl, hid, 1, w.num_blocks, two.k, two.v), "append")
    want = two.decode([0])
    got = one.new_out()
    ps, ph = torch.arange(len(lens), device=DEV).int(), torch.zeros(len(lens), dtype=torch.int32, device=DEV)
    H.check(H.hetis_attn_decode_pairs_step_ws(one.shape, one.q, kn, vn, one.k.view(-1, 16, D), one.v.view(-1, 16, D),
                                              one.bt, one.sl, ps, ph, len(lens), one.scale, got, ws, ws.numel()), "step")
    torch.cuda.synchronize()
    no_expired_wait(ws)
    assert way(ws) == expected
    same = lambda a, b: torch.equal(a.view(torch.int16), b.view(torch.int16))
    assert same(one.k, two.k) and same(one.v, two.v) and same(got, want)


@pytest.mark.parametrize("Hq,D", [(1, 64), (1, 128), (2, 64), (2, 128), (4, 64), (4, 128), (8, 64), (8, 128)])
@pytest.mark.parametrize("edge", [0, -1, 1])
def test_edges_of_pieces_and_windows(Hq, D, edge):
    """Rows that end at, just before and just behind a tile, a piece, a window, a segment."""
    piece = 128 if Hq >= 4 else 64
    ends = [16, piece, 2 * piece, 3 * piece, 4 * piece, 5 * piece, 1024, 1024 + piece, 4096 - 4 * piece, 4096, 4096 + piece]
    compare([max(0, e + edge) for e in ends], Hq, D, TEAM_ITEMS)


@pytest.mark.parametrize("Hq,D", [(1, 128), (2, 64), (4, 128), (8, 64)])
@pytest.mark.parametrize("rows,windows", [(64, 4), (51, 5), (52, 5), (85, 3), (86, 3), (255, 1), (256, 1), (257, 1)])
def test_as_many_items_as_workgroups(Hq, D, rows, windows):
    """One item a workgroup and one more, rows of one length and ragged: teams on items of a row, on whole rows of
    one item, and on neither side of the line."""
    window = 512 if Hq >= 4 else 256
    if windows > 1:
        expected = TEAM_ITEMS if rows * windows <= 256 else CHUNKS
    else:
        expected = TEAM_ROWS if rows <= 256 else WAVE_ROWS
    compare([windows * window] * rows, Hq, D, expected)
    compare([windows * window - 7 * (i % 11) for i in range(rows)], Hq, D, expected)


@pytest.mark.parametrize("r,D", [(1, 64), (2, 128), (4, 64), (8, 128)])
@pytest.mark.parametrize("B,lens,expected", [
    (21, (600, 900), TEAM_ROWS),        # x 12 heads: 252 rows that keep most of the chip busy
    (4, (700, 1200), TEAM_ITEMS),       # 48 rows of several items
    (2, (100, 2500), TEAM_ITEMS),
    (3, (9000, 12000), CHUNKS),         # more items than workgroups
])
def test_teams_on_several_heads(r, D, B, lens, expected):
    """Rows of 12 selected heads, in an order of their own: against the checker, and one of them alone, bit for bit."""
    rng = np.random.default_rng(B)
    lens = rng.integers(lens[0], lens[1] + 1, size=B)
    Hkv, sel = 14, [13, 0, 7, 1, 12, 4, 6, 5, 9, 8, 2, 11]
    w = W.make_custom([int(x) for x in lens], Hkv * r, Hkv, D, sel, seed=B + r, device=DEV, max_seq_len=12000)
    d = Dev(w)
    ws = d.workspace(len(sel))
    out = d.decode_ws(sel, ws)
    assert way(ws) == expected
    ref = oracle.attn_decode(w.q.cpu().numpy(), w.k_cache.cpu().numpy(), w.v_cache.cpu().numpy(), w.block_table,
                             w.seq_lens, np.asarray(sel, dtype=np.int32), w.spec.scale)
    check_rows(out, ref, selected_rows(w.spec, sel), TOL, "team of several heads")
    one = d.decode_ws([7], d.workspace(1))
    rows = slice(7 * r, 8 * r)
    assert np.array_equal(bits(out)[:, rows], bits(one)[:, rows])
    no_expired_wait(ws)
