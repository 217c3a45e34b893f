"""Rows around whole turns of a wave's ring of tiles.  The ring is one tile pair deep (two at 64
dims) in launches of many rows and twice that in launches of few rows and in split calls; every
kind of launch gives the same rows the same bits, and all agree with the checker."""
import numpy as np
import pytest

import oracle
from paper_2509_08309_amd import workloads as W

from gpu_harness import TOL, Dev, bits, check_rows, no_expired_wait, selected_rows

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LENS = [0, 1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 80, 81, 95, 96, 97, 127, 128, 129, 160, 192, 255, 256,
        257, 288, 320, 500, 1023, 1024, 1025, 1100, 2047, 4096]


@pytest.mark.parametrize("r,D", [(1, 64), (1, 128), (2, 64), (2, 128), (4, 128), (8, 64)])
def test_turns_of_the_ring(r, D):
    Hkv, few, some = 32, [30, 2, 17], list(range(1, 21)) + [30]
    w = W.make_custom(LENS, Hkv * r, Hkv, D, few, seed=10 * D + r, device=DEV)
    d = Dev(w)
    out = d.decode(few)                         # 108 rows: single chunks, or one row a workgroup
    ref = oracle.attn_decode(w.q.cpu().numpy(), w.k_cache.cpu().numpy(), w.v_cache.cpu().numpy(),
                             w.block_table, w.seq_lens, np.asarray(few, dtype=np.int32), w.spec.scale)
    rows = selected_rows(w.spec, few)
    check_rows(out, ref, rows, TOL, "few rows")
    every = d.decode(list(range(Hkv)))          # 1152 rows: whole segments by ticket
    assert np.array_equal(bits(out)[:, rows], bits(every)[:, rows])
    mid = d.decode(some)                        # 756 rows: fixed second and third segments
    rows_mid = selected_rows(w.spec, some)
    assert np.array_equal(bits(mid)[:, rows_mid], bits(every)[:, rows_mid])
    for chunk in (16, 32, 48, 256):             # 108 and 756 rows of single chunks
        o_p, lse_p = d.split(few, chunk, max(LENS))
        check_rows(d.merge(o_p, lse_p, few, chunk, max(LENS)), ref, rows, TOL, f"split {chunk}")
        o_m, lse_m = d.split(some, chunk, max(LENS))
        both = [some.index(30), some.index(2), some.index(17)]
        assert np.array_equal(o_p.cpu().numpy().view(np.int32), o_m[:, both].cpu().numpy().view(np.int32))
        assert np.array_equal(lse_p.cpu().numpy().view(np.int32), lse_m[:, both].cpu().numpy().view(np.int32))
    no_expired_wait()
