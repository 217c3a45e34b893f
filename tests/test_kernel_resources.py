"""What the compiler made of the kernels, checked without a GPU: no kernel of the library may use
scratch (private) memory.  In the Attention kernel a scratch store sits in a streaming wave,
where any store makes the waits on the tile loads inexact (a struct with padding bytes or a
small array of HIP's vector structs is enough for the compiler to produce one); in the cache
kernels it would double the traffic.  Also: register counts within what two waves per SIMD
allow (the Attention kernel's workgroup has five waves on four SIMDs)."""
import functools
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2509_08309_amd import build

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@functools.lru_cache(maxsize=None)
def assembly(source):
    with tempfile.TemporaryDirectory() as d:
        asm = os.path.join(d, source + ".s")
        flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
        subprocess.run([HIPCC] + flags + ["-S", "--cuda-device-only", "-o", asm,
                                          os.path.join(build.CSRC, source)], check=True,
                       stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
        with open(asm) as f:
            return f.read()


def kernel_metadata(source):
    text = assembly(source)
    meta = {}
    for m in re.finditer(r"\.name:\s+(\S+)\n((?:\s+\.\w+:.*\n)+)", text):
        fields = dict(re.findall(r"\.(\w+):\s+(\S+)", m.group(2)))
        if "vgpr_count" in fields:
            meta[m.group(1)] = fields
    return meta


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
@pytest.mark.parametrize("source,expected", [("hetis_attn.hip", 64 + 16), ("hetis_kv.hip", 8)])
def test_no_kernel_uses_scratch_memory(source, expected):
    meta = kernel_metadata(source)
    main = {k: v for k, v in meta.items() if "persistent_kernel" in k or "wave_rows_kernel" in k or "kv_" in k}
    assert len(main) == expected, sorted(meta)
    for name, f in meta.items():
        assert int(f["private_segment_fixed_size"]) == 0, (name, f["private_segment_fixed_size"])
        assert int(f.get("vgpr_spill_count", 0)) == 0, name
        assert int(f["vgpr_count"]) + int(f.get("agpr_count", 0)) <= 256, (name, f["vgpr_count"])


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
def test_registers_of_the_combination_of_four_rows():
    """The combination of partial results shares the streaming loop's kernel: with four query rows a
    batch of them may not take the kernel to the limit of 256 registers."""
    meta = kernel_metadata("hetis_attn.hip")
    for dim, limit in ((64, 190), (128, 244)):
        mine = [f for k, f in meta.items() if re.search(rf"MfmaPolicyILi{dim}ELi4E.*Li2EEEv", k)]
        assert len(mine) == 2                       # common subset, pairs
        for f in mine:
            assert int(f["vgpr_count"]) <= limit, f["vgpr_count"]


def streaming_loops(policy, dim, group, variant):
    """Loops of the persistent kernel (both forms) that ask for the tiles of one turn of the ring, as lists of
    instructions: innermost, without a call for block ids or for the next chunk."""
    text, out = assembly("hetis_attn.hip"), []
    names = re.findall(rf"^(\S*persistent_kernel\S*{policy}PolicyILi{dim}ELi{group}E\S*Li{variant}EEEv\S*):", text, re.M)
    assert len(names) == 2, names
    for name in names:
        start = text.index("\n" + name + ":")
        lines = text[start:text.index(".Lfunc_end", start)].split("\n")
        at = {l.split(":")[0]: i for i, l in enumerate(lines) if l.startswith(".LBB")}
        spans = {}
        for i, l in enumerate(lines):
            s = l.split()
            if s and s[0].startswith(("s_cbranch", "s_branch")) and at.get(s[1], i) < i:
                spans[at[s[1]]] = i                             # the whole loop: its last branch back
        for a, b in spans.items():
            body = [l.strip() for l in lines[a:b] if l.startswith("\t") and l.strip()[0] not in ".;"]
            inner = any(a < c and spans[c] <= b for c in spans)
            if not inner and not any(x.startswith(("s_load", "ds_")) for x in body) and \
                    any(x.startswith("buffer_load_dwordx4") for x in body):
                out.append(body)
    return out


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
@pytest.mark.parametrize("dim,group", [(64, 1), (64, 2), (128, 1), (128, 2)])
def test_a_piece_is_folded_in_place(dim, group):
    """What the fold of a piece costs a wave: the state's registers are scaled and summed where they are, so that
    the only moves of a turn are the zeros that the next piece starts from (ten a query row) and those of the
    tiles' arithmetic, the zeros that its dot products start from."""
    for b in [b for v in (0, 1, 2) for b in streaming_loops("Vec", dim, group, v)]:
        moves = sum(x.startswith("v_mov_b32") for x in b)
        scores = sum(x.startswith("buffer_load") for x in b) // 2 * group
        assert moves <= 10 * group + scores + 6, (len(b), moves, scores)


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
@pytest.mark.parametrize("policy,dim,group", [("Vec", 128, 1), ("Vec", 64, 2), ("Mfma", 128, 8)])
def test_launches_without_teams_carry_no_team_code(policy, dim, group):
    """The instantiation for more rows than workgroups is the smaller one by the team's code."""
    text = assembly("hetis_attn.hip")
    size = {}
    for m in re.finditer(rf"^(\S*persistent_kernel\S*{policy}PolicyILi{dim}ELi{group}E\S*Lb0ELi([23])EEEv\S*):", text, re.M):
        size[m.group(2)] = int(re.search(r"codeLenInByte = (\d+)", text[m.end():]).group(1))
    assert size["3"] > 1.15 * size["2"], size


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not found")
@pytest.mark.parametrize("dim,group,variant", [(d, g, v) for d in (64, 128) for g in (1, 2) for v in (0, 1, 2, 3)
                                               if (d, g, v) != (64, 1, 3)])      # drained on purpose
def test_a_turn_of_the_ring_does_not_drain_it(dim, group, variant):
    """Vector path: a slot is refilled as soon as its tile is used, so what a turn waits for ahead of its first
    refill is that tile, not the whole ring."""
    a_tile = dim // 16                                      # loads of a K tile and a V tile
    for b in streaming_loops("Vec", dim, group, variant):
        loads = sum(x.startswith("buffer_load") for x in b)
        ahead = b[:next(i for i, x in enumerate(b) if x.startswith("buffer_load"))]
        left = [int(re.search(r"vmcnt\((\d+)\)", x).group(1)) for x in ahead if "vmcnt" in x][-1]
        assert left >= loads - a_tile, (len(b), loads, left)
