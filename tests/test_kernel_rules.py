"""Rules of the Attention kernel that do not show in a result, checked at compile time: the headers
are compiled on the host with the rule as a static_assert."""
import os
import shutil
import subprocess

import pytest

from paper_2509_08309_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")


def assert_compiles(tmp_path, body):
    src = tmp_path / "rule.hip"
    src.write_text('#include "attn_mfma.hpp"\n#include "attn_vec.hpp"\nusing namespace hetis;\n' + body)
    r = subprocess.run([HIPCC, "-std=c++17", "--offload-arch=gfx950", "--cuda-host-only", "-fsyntax-only",
                        "-I", build.CSRC, str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


@pytest.mark.parametrize("R", [1, 2])
@pytest.mark.parametrize("D", [64, 128])
def test_depth_of_the_ring_follows_the_rows(tmp_path, D, R):
    """Few rows deep; many rows deep when most are of 2 (64 dims: 3) to 8 tiles.  No other argument:
    what the block table allows has no say."""
    ring = 2 if D == 64 else 1
    P = f"VecPolicy<{D}, {R}>"
    assert_compiles(tmp_path, f"""
        static_assert({P}::ring(false) == {ring} && {P}::ring(true) == {2 * ring}, "8 and 16 KB");
        static_assert(deep_ring<{P}>(1, 0) && deep_ring<{P}>(511, 0), "few rows");
        static_assert(!deep_ring<{P}>(512, 0) && !deep_ring<{P}>(1 << 21, 39), "many rows");
        static_assert(deep_ring<{P}>(512, 40) && deep_ring<{P}>(1 << 21, 64), "many short rows");
        static_assert(!short_row<{P}>(0) && !short_row<{P}>({16 * ring}) && !short_row<{P}>(129) &&
                      !short_row<{P}>(-5) && !short_row<{P}>(4096) && !short_row<{P}>(1 << 30), "not short");
        static_assert(short_row<{P}>({16 * ring + 1}) && short_row<{P}>(128), "short");
    """)


def test_bound_of_a_wait_is_a_time(tmp_path):
    """However often a wait looks, it gives up after 2^30 cycles of sleep, not earlier."""
    assert_compiles(tmp_path, """
        static_assert(kPollSleep >= 1 && 64ll * kPollSleep * kSpinLimit >= (1ll << 30) - 64ll * kPollSleep &&
                      64ll * kPollSleep * kSpinLimit <= 1ll << 30, "0.4 s");
    """)


def test_one_instantiation_holds_split_calls(tmp_path):
    """Both sides of the kernel and the host's check go by the same predicate."""
    assert_compiles(tmp_path, """
        static_assert(holds_split(kVariantPlain, false), "split calls run here");
        static_assert(!holds_split(kVariantPlain, true) && !holds_split(kVariantFew, false) &&
                      !holds_split(kVariantFew, true) && !holds_split(kVariantMerge, false) &&
                      !holds_split(kVariantMerge, true), "and nowhere else");
    """)
    with open(os.path.join(build.CSRC, "attn_persist.hpp")) as f:
        kernel = f.read()
    assert kernel.count("p.mode == kModeSplit") == 1, "one place decides: split_mode"
    with open(os.path.join(build.CSRC, "hetis_attn.hip")) as f:
        assert "!holds_split(variant, pairs)) return HETIS_ERR_UNSUPPORTED;" in f.read()


def test_teams_are_compiled_in_where_they_can_run(tmp_path):
    """No more rows than workgroups, in a launch that may be handed out singly; its code is in no other
    instantiation."""
    assert_compiles(tmp_path, """
        static_assert(merge_variant(kModeSpread, 1, 256) == kVariantTeam && merge_variant(kModeSpread, 256, 256) == kVariantTeam);
        static_assert(merge_variant(kModeSpread, 257, 256) == kVariantMerge && merge_variant(kModeSpread, 511, 256) == kVariantMerge);
        static_assert(merge_variant(kModeSegments, 1, 256) == kVariantMerge && merge_variant(kModeSegments, 4096, 256) == kVariantMerge);
        static_assert(!holds_split(kVariantTeam, false) && !holds_split(kVariantTeam, true));
    """)


@pytest.mark.parametrize("first,last", [(1, 8), (8, 64), (64, 200), (200, 350), (350, 512)])
def test_division_by_a_multiplication(tmp_path, first, last):
    """divide_by over every divisor of a launch of few rows: the quotient changes at the multiples and nowhere
    else, up to the largest item number."""
    assert_compiles(tmp_path, f"""
        constexpr bool exact() {{
            for (unsigned n = {first}; n < {last}; ++n) {{
                const unsigned i = inverse_of(n);
                for (unsigned q = 0; q * n < 8192; ++q)
                    if (divide_by(q * n, i) != q || divide_by(q * n + n - 1, i) != q) return false;
                if (divide_by(8191, i) != 8191 / n) return false;
            }}
            return true;
        }}
        static_assert(exact(), "as / has it");
    """)


@pytest.mark.parametrize("R", [4, 8])
def test_depth_of_the_ring_on_the_mfma_path(tmp_path, R):
    """16 KB of tiles a wave with 64 dims, 24 KB with 128, in decode calls of every size; less in split calls."""
    assert_compiles(tmp_path, f"""
        static_assert(MfmaPolicy<64, {R}>::ring(true) == 4 && MfmaPolicy<64, {R}>::ring(false) == 4, "16 KB");
        static_assert(MfmaPolicy<128, {R}>::ring(true) == 3 && MfmaPolicy<128, {R}>::ring(false) == 3, "24 KB");
        static_assert(MfmaPolicy<64, {R}>::ring_split == 3 && MfmaPolicy<128, {R}>::ring_split == 2, "12 and 16 KB");
        static_assert(VecPolicy<64, 1>::ring_split == VecPolicy<64, 1>::ring(true) &&
                      VecPolicy<128, 2>::ring_split == VecPolicy<128, 2>::ring(true), "the deep one");
    """)
