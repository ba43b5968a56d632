"""Registers and LDS of the layer kernel's variants, from the metadata the compiler wrote into the built library: what only link
scores need must not crowd the variants that every streamed batch runs."""
import os
import re
import struct
import subprocess

import pytest

from paper_2603_21090_amd import binding

READELF = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath("/opt/rocm/bin/hipcc"))), "llvm", "bin", "llvm-readelf")
# key slots, time slots, raw edge rows, heads, ring entries per chunk, workgroups per CU, delta, query cache, root nodes
VARIANT = re.compile(r"layer_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)ELi(\d)ELb(\d)ELb(\d)E(?:Lb(\d)E)?E")


@pytest.fixture(scope="module")
def notes(tmp_path_factory):
    """name of a layer kernel -> (spilled vector registers, bytes of LDS of its own, bytes of scratch memory a lane)"""
    if not os.path.exists(binding.LIB_PATH):
        from paper_2603_21090_amd import build
        build.build_library()
    blob = open(binding.LIB_PATH, "rb").read()
    magic, out, at = b"__CLANG_OFFLOAD_BUNDLE__", {}, 0
    while (at := blob.find(magic, at)) >= 0:
        p = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", blob, p - 8)[0]):
            off, size, n = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" not in triple or size == 0:
                continue
            obj = tmp_path_factory.mktemp("objects") / f"{len(out)}.o"
            obj.write_bytes(blob[at + off:at + off + size])
            text = subprocess.run([READELF, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
            for block in re.split(r"\n  - ", text):            # (a kernel's entry)
                if (name := re.search(r"\.name:\s+(\S*layer\w*_kernel\S*)", block)):
                    out[name[1]] = tuple(int(re.search(rf"\.{field}:\s+(\d+)", block)[1])
                                         for field in ("vgpr_spill_count", "group_segment_fixed_size", "private_segment_fixed_size"))
        at += len(magic)
    return out


@pytest.fixture(scope="module")
def spills(notes):
    """variant -> spilled vector registers"""
    return {tuple(int(x or 0) for x in m.groups()): n for name, (n, _, _) in notes.items() if (m := VARIANT.search(name))}


@pytest.mark.parametrize("qcache", [0, 1])
@pytest.mark.parametrize("raw_edges", [0, 1])
@pytest.mark.parametrize("heads", [1, 2])
@pytest.mark.parametrize("time_slots", [1, 2])
def test_streamed_variants_of_two_key_slots(spills, time_slots, heads, raw_edges, qcache):
    """Rows of up to 128 floats in two slots: nothing spilled."""
    variant = (2, time_slots, raw_edges, heads, 1, 2, 0, qcache)
    assert spills[variant + (0,)] == 0


def test_streamed_variants_of_one_and_four_key_slots(spills):
    """Rows of one slot: nothing spilled; of four, whose waves use all 128 registers: four at most."""
    streamed = {v: n for v, n in spills.items() if not v[6] and not v[8]}
    assert {v[0] for v in streamed} == {1, 2, 4}
    for v, n in streamed.items():
        assert n <= (4 if v[0] == 4 else 0), v


def test_link_scores_have_variants_of_their_own(spills):
    streamed = {v[:8] for v in spills if not v[6] and not v[8]}
    assert streamed and streamed == {v[:8] for v in spills if v[8]}


def test_the_launches_allow_for_the_kernels_own_lds(notes):
    """Launches fit their tiles into what 3,072 bytes leave of a workgroup's share of the LDS (kFixedLds).  A kernel with two bodies
    once held its arrays twice, 4,560 bytes: rows of 22 to 24 entries then had one workgroup per CU instead of two."""
    assert any("layer32_kernel" in name for name in notes)
    for name, (_, lds, _) in notes.items():
        assert 0 < lds <= 3072, name


def test_delta_variants(spills):
    """One slot (168 registers): one spilled at most; two: none; four, eight in the widest."""
    delta = {v: n for v, n in spills.items() if v[6]}
    assert {v[0] for v in delta} == {1, 2, 4}
    for v, n in delta.items():
        assert n <= {1: 1, 2: 0, 4: 8}[v[0]], v


def test_nothing_but_spilled_registers_lies_in_scratch_memory(notes):
    """What a kernel keeps in scratch memory of its own will is a store and a load in front of what it is for (a flag of the products'
    groups was, once per chunk, with raw edge rows)."""
    for name, (spilled, _, scratch) in notes.items():
        assert spilled or not scratch, (name, scratch)


def test_variants_of_long_lists(notes):
    """Kernels of 32-row tiles: nothing spilled without the query cache.  With it, where a tile holds the next one's rows through its last
    two phases, a pair of registers in the widest models of two slots and up to four registers with four slots, reloaded once a tile;
    none of them a constant of a division, whose reload waited for the weights requested ahead of it."""
    name = re.compile(r"layer32_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELb(\d)E")
    tall = {tuple(map(int, m.groups())): n for key, (n, _, _) in notes.items() if (m := name.search(key))}
    assert {(v[0], v[4]) for v in tall} == {(2, 0), (2, 1), (4, 0), (4, 1)}
    for v, n in tall.items():
        assert n <= (0 if not v[4] else 2 if v[0] == 2 else 4), v
    assert tall[2, 2, 0, 2, 1] == 0                            # (heads of 33 to 64 floats, wide edge features: the common shape)
