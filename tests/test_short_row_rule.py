"""Which launches give a wave a row (row_a_wave), on both sides of its lines: rows, compute units, tokens a row of
the block table holds."""
import shutil

import pytest

from test_kernel_rules import HIPCC, assert_compiles

pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")


@pytest.mark.parametrize("D,R", [(D, R) for D in (64, 128) for R in (1, 2, 4, 8)])
def test_lines(tmp_path, D, R):
    piece, chunk = (128, 512) if R >= 4 else (64, 256)
    mid = 384 if R == 2 or (D, R) == (64, 8) else 512            # fewer rows than SIMDs
    lines = [(1, piece), (256, piece), (257, chunk), (511, chunk), (512, mid), (1023, mid), (1024, 512), (2048, 512),
             (2049, 384), (65535 * 1024, 384)]
    body = "".join(f"static_assert(row_a_wave<{D}, {R}>({n}, 256, {t}) && !row_a_wave<{D}, {R}>({n}, 256, {t + 16}));\n"
                   for n, t in lines)
    assert_compiles(tmp_path, '#include "attn_rows.hpp"\n' + body)
