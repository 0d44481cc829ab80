"""Registers and LDS of the streaming decode kernels, read from the built library's own code-object metadata (no GPU):
the forms that run 256 workgroups of eight wavefronts per row need several of them on a CU at a time."""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

import paper_2404_01365_amd as G

LIB = os.path.join(os.path.dirname(G.__file__), "libgriffin.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _notes(elf):
    """msgpack metadata of an amdgpu code object (note type 32)"""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        typ, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
        if typ != 7:
            continue
        namesz, descsz, ntype = struct.unpack_from("<III", elf, off)
        if ntype == 32:
            start = off + 12 + (namesz + 3) // 4 * 4
            return msgpack.unpackb(elf[start:start + descsz])
    return {}


def kernels():
    blob = open(LIB, "rb").read()
    found = {}
    for m in re.finditer(MAGIC, blob):
        base = m.start()
        count, = struct.unpack_from("<Q", blob, base + len(MAGIC))
        at = base + len(MAGIC) + 8
        if count > 8:
            continue
        for _ in range(count):
            off, size, tlen = struct.unpack_from("<QQQ", blob, at)
            triple = blob[at + 24:at + 24 + tlen]
            at += 24 + tlen
            if b"gfx950" in triple:
                for k in _notes(blob[base + off:base + off + size]).get("amdhsa.kernels", []):
                    found[k[".name"]] = k
    return found


# template arguments as the compiler mangles them: <BF16, GATED, INDEXED, BIAS, rows>, <BF16, GATED, BIAS> of the per-row blocks
def name(kernel, *flags, rows=None):
    args = "".join("Lb%dE" % f for f in flags) + ("" if rows is None else "Li%dE" % rows)
    return r"%sI%sE" % (kernel, args)


@pytest.mark.parametrize("pattern,vgprs", [
    (name("ff_decode_kernel", 1, 1, 1, 0, rows=1), 80),        # own sets, bf16 Eq. 3: six waves a SIMD, three workgroups a CU
    (name("ff_decode_kernel", 1, 0, 1, 0, rows=1), 72),        # ... Eq. 2
    (name("ff_decode_kernel", 0, 1, 1, 1, rows=1), 72),        # ... fp32 with biases
    (name("ff_decode_multi_kernel", 1, 1, 1), 80),             # per-row blocks, bf16 Eq. 3 with biases
    (name("ff_decode_multi_kernel", 1, 0, 1), 64),             # ... Eq. 2: eight waves a SIMD, four workgroups a CU
    (name("ff_decode_kernel", 1, 1, 0, 1, rows=1), 80),        # one row through one block, with biases
])
def test_rows_that_go_alone_keep_their_occupancy(pattern, vgprs):
    hits = [k for n, k in kernels().items() if re.search(pattern, n)]
    assert len(hits) == 1, pattern
    k = hits[0]
    assert k[".vgpr_count"] <= vgprs
    assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0
    assert k[".group_segment_fixed_size"] <= 40 * 1024         # four workgroups a CU


# fp32 product <ACT, GATED, BBF16, VEC>, 16-token tiles.  What its loop takes with the loads in the order of the source: where a load was made
# zero at once the compiler moved them (160 instead of 148, 144 and 145, 96 instead of 85), and calls were 1 to 3 % slower
@pytest.mark.parametrize("flags,tiles,vgprs", [((1, 1, 0, 1), 2, 150), ((1, 1, 0, 1), 4, 248), ((1, 0, 0, 1), 2, 88), ((1, 0, 0, 1), 4, 148),
                                               ((0, 0, 0, 1), 2, 88), ((0, 0, 0, 1), 4, 148), ((0, 0, 1, 1), 2, 88), ((0, 0, 1, 1), 4, 148)])
def test_fp32_product_keeps_its_registers(flags, tiles, vgprs):
    hits = [k for n, k in kernels().items() if re.search("f32_nt_kernelI%sLi%dELi1E" % ("".join("Lb%dE" % f for f in flags), tiles), n)]
    assert len(hits) == 1 and hits[0][".vgpr_count"] <= vgprs and hits[0][".private_segment_fixed_size"] == 0


@pytest.mark.parametrize("bf16", [0, 1])
@pytest.mark.parametrize("gated", [0, 1])
def test_rows_that_go_four_at_a_time_leave_room_for_three_workgroups(bf16, gated):
    for bias in (0, 1):
        hits = [k for n, k in kernels().items() if re.search(name("ff_decode_kernel", bf16, gated, 0, bias, rows=4), n)]
        assert len(hits) == 1 and hits[0][".group_segment_fixed_size"] <= 48 * 1024


def test_forms_of_the_prompt_product_keep_their_registers():
    """One wave a SIMD: nothing in scratch but for the largest tile of an Eq. 2 block.  Raw products of 64 tokens go two workgroups a CU."""
    import launches
    seen = two = 0
    for n, k in kernels().items():
        if launches.two_shapes(n):
            two += 1
            assert k[".private_segment_fixed_size"] == 0 and k[".group_segment_fixed_size"] <= 160 * 1024, n
        form = launches.form(n)
        if form is None:
            continue
        seen += 1
        assert k[".private_segment_fixed_size"] <= (64 if form == "256x256 Eq. 2" else 0), n
        assert k[".group_segment_fixed_size"] <= 160 * 1024
        if form in ("64x128 raw Eq. 3", "64x256 raw one matrix"):
            assert k[".vgpr_count"] <= 256 and k[".group_segment_fixed_size"] <= 80 * 1024
    assert seen == 121                   # 37 of each activation and ten raw products
    assert two == 24                     # four heights, with a copy and without, of each activation


def test_selection_kernels_stay_out_of_scratch():
    """... but for two words of a top-k of 32 scores a thread, on its own and beside other work; and workgroups of sixteen waves, two of them a CU."""
    found = {n: k for n, k in kernels().items() if re.search("topk_reg_kernel|topk_kernel|stat_whole_kernel", n)}
    assert len(found) == 8 + 4 + 4 * 8 + 2
    for n, k in found.items():
        assert k[".private_segment_fixed_size"] <= (8 if "Li32E" in n else 0), n
        assert k[".group_segment_fixed_size"] <= 80 * 1024 and k[".vgpr_count"] <= (64 if "stat_whole" in n else 128), n
