"""Which form of the prompt product a call takes, and what it makes of it (no GPU: tests/launches.py)."""
import ctypes
import re

import pytest

import launches
import paper_2404_01365_amd as G
import test_gpu_parity as cases
import test_kernel_resources as resources


def routes(calls):
    return [[launches.route(l) for l in ls if launches.form(l["name"])] for ls in launches.record(calls)]


# d, D_ff, tokens of an Eq. 3 block whose products are summed in parts; the form, and sums kept apart in registers (1: ranges with slabs)
PARTS = [
    (4096, 11008, 40, "64x64 Eq. 3 copy", 4),
    (4608, 21712, 316, "128x128 Eq. 3", 2),
    (3648, 9488, 196, "224x128 raw Eq. 3", 1),        # not 75 x 2 tiles of 256 x 64
    (1728, 3456, 585, "256x64 Eq. 3 copy", 3),
    (4416, 15856, 220, "256x64 Eq. 3 copy", 2),
    (6144, 16288, 100, "128x128 raw Eq. 3", 1),       # not one row of 128 x 64
    (3072, 8176, 196, "128x64 Eq. 3 copy", 4),
    (8128, 12304, 108, "128x64 Eq. 3 copy", 5),
    (2560, 17424, 47, "64x128 raw Eq. 3", 1),         # not 128 x 128 of which 47 tokens are there
    (3072, 22800, 1, "64x128 raw Eq. 3", 1),
    (3584, 19536, 57, "128x128 Eq. 3", 2),
    (1536, 3072, 3, "64x128 raw Eq. 3", 1),           # not 48 tiles of 64 x 64
    (1536, 4176, 3, "64x64 Eq. 3 copy", 6),
]


def test_sums_stay_apart_in_registers_only_where_that_is_faster():
    got = routes([dict(entry="select", d=d, n=F, lens=[S]) for d, F, S, *_ in PARTS])
    assert [(*c[:3], r[0][0], r[0][3]) for c, r in zip(PARTS, got)] == PARTS


@pytest.mark.parametrize("act", [G.ACT_SILU, G.ACT_GELU_TANH, G.ACT_RELU])
@pytest.mark.parametrize("ti,ni,gated,wide", [(5, 4, 1, 0), (8, 1, 1, 0), (0, 0, 1, 0), (8, 2, 0, 1), (6, 2, 0, 1), (8, 3, 0, 0), (6, 4, 0, 0)])
def test_a_shape_that_is_not_compiled_is_refused(act, ti, ni, gated, wide):
    """The rule that chooses shapes and the list of those compiled are apart: a launch of nothing must not look like success."""
    launch = getattr(G.lib, "_ZN7griffin16launch_ff1_tilesILi%dEEEiRKNS_9Ff1ParamsEiibbiP12ihipStream_t" % act)
    launch.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.c_bool, ctypes.c_int, ctypes.c_void_p]
    p = launches.Ff1Params()
    assert launch(ctypes.byref(p), ti, ni, bool(gated), bool(wide), 8, None) == G.EUNSUPPORTED


def test_the_gpu_cases_reach_every_form_as_they_say():
    calls = [dict(entry="select", d=d, n=F, lens=[S], act=act, gated=gated, bias=bias) for d, F, S, act, gated, bias, *_ in cases.FORM_CASES]
    calls += [dict(entry="phase", d=d, n=F, lens=[S]) for d, F, S, *_ in cases.FORM_PHASE_CASES]
    calls += [dict(entry="out", d=d, n=F, lens=[S]) for d, F, S, *_ in cases.FORM_OUT_CASES]
    listed = [c[6:] for c in cases.FORM_CASES] + [c[3:] for c in cases.FORM_PHASE_CASES] + [(*c[3:], 1) for c in cases.FORM_OUT_CASES]
    got = [r[0] for r in routes(calls)]
    assert [(c, r) for c, r in zip(calls, got) if r not in listed] == []
    assert got == listed
    # ... and the second product of a prompt phase, and outputs of few tokens, in the lists that have been there
    got += [r for rs in routes([dict(entry="out", d=d, n=F, lens=[S]) for d, F, S in ((4200, 320, 6000), (2048, 128, 300), (131404, 128, 5))]) for r in rs]
    compiled = {launches.form(n) for n in resources.kernels()} - {None}
    assert compiled - {r[0] for r in got} == set()
    for form in compiled:
        _, tiles, kts, sums = zip(*(r for r in got if r[0] == form))
        deep = form.startswith(("64x64", "96x64", "128x64", "64x128 Eq. 2"))       # four stages or more
        assert max(kts) >= (8 if deep else 5), form


def test_the_least_workspace_takes_tiles_of_128_neurons():
    calls = [dict(entry=e, d=64, n=16576, lens=[399], least=least) for e in ("select", "phase") for least in (False, True)]
    assert [r[0][0] for r in routes(calls)] == ["256x96 Eq. 3", "192x128 Eq. 3", "256x96 Eq. 3 copy", "192x128 Eq. 3 copy"]
    calls = [dict(entry="select", d=1024, n=1000, lens=[40], least=least) for least in (False, True)]
    assert [r[0][::3] for r in routes(calls)] == [("64x64 Eq. 3 copy", 4), ("128x128 Eq. 3", 1)]


def dealt(tiles_a, tiles_b, workgroups):
    """The tiles of both shapes that each workgroup of ff1_bf16_two_shapes_kernel takes, by its own rule."""
    for wg in range(workgroups):
        x, slot, per = wg % 8, wg // 8, workgroups // 8
        a0, a1 = x * tiles_a // 8, (x + 1) * tiles_a // 8
        b0, b1 = x * (tiles_a + tiles_b) // 8 - a0, (x + 1) * (tiles_a + tiles_b) // 8 - a1
        yield list(range(a0 + slot, a1, per)), list(range(b0 + per - 1 - slot, b1, per))


def test_products_on_two_shapes_cover_the_block_once():
    two = cases.TWO_SHAPES_CASES
    calls = [dict(entry="phase" if ph else "select", d=d, n=F, lens=[S], act=act if not ph else G.ACT_SILU) for d, F, S, act, ph, *_ in two]
    walked = 0
    for c, ls in zip(two, launches.record(calls)):
        first = [l for l in ls if launches.two_shapes(l["name"])]
        assert len(first) == 1 and not any(launches.form(l["name"]) and " raw " not in launches.form(l["name"]) for l in ls), c
        act, copy, shape_a, shape_b = launches.two_shapes(first[0]["name"])
        l, b, (d, F, S, want, ph, height, wide, narrow) = first[0], first[0]["second"], c
        assert (shape_a, shape_b, copy, act) == ((height, 128), (height, 96), ph, G.ACT_SILU if ph else want), c
        assert l["nt"] == wide and l["F"] == min(F, 128 * wide) and l["mt"] == -(-S // height), c
        # the second part: the neurons that follow, their rows of the weights, columns of Z and of its copy, and row sums
        assert b["F"] == F - l["F"] and b["nt"] == narrow == -(-b["F"] // 96), c
        at = {"W1": 2 * l["ldw"] * l["F"], "Wg": 2 * l["ldw"] * l["F"], "Z": 4 * l["F"], "rowpart": 4 * wide, "Zb": 2 * l["F"] if copy else 0}
        assert {f: b[f] - l[f] for f in at} == at, c
        assert all(b[f] == l[f] for f in ("X", "ldx", "ldw", "ldz", "ldzb", "M", "d", "mt", "splits", "kt_per_split", "kt_per_sum", "z_stream", "rotate", "nt_row"))
        assert l["nt_row"] == wide + narrow and l["splits"] == 1 and l["kt_per_split"] == d // 64, c
        # every tile of both is dealt once
        tiles_a, tiles_b = l["mt"] * wide, l["mt"] * narrow
        assert l["grid"][0] % 8 == 0 and l["grid"][1:] == [1, 1]
        shares = list(dealt(tiles_a, tiles_b, l["grid"][0]))
        assert sorted(t for a, _ in shares for t in a) == list(range(tiles_a)) and sorted(t for _, b_ in shares for t in b_) == list(range(tiles_b)), c
        walked += max(len(a) for a, _ in shares) > 1 and max(len(b_) for _, b_ in shares) > 1 and l["mt"] > 8
    assert walked >= 3             # cases where a workgroup walks several tiles of both, over more than one panel


def test_two_shapes_need_room_for_their_row_sums_and_a_lean_block():
    d, F, S = 768, 16756, 683
    names = lambda **kw: [l["name"] for l in launches.record([dict(dict(entry="select", d=d, n=F, lens=[S]), **kw)])[0]]  # noqa: E731
    assert any("two_shapes" in n for n in names())
    for kw in (dict(least=True), dict(bias=True), dict(gated=False), dict(d=704), dict(dtype=G.F32)):
        assert not any("two_shapes" in n for n in names(**kw)), kw


def test_statistic_in_one_kernel_while_a_cu_reads_little():
    calls = [(4096, 11008, [512]), (1024, 11008, [1500]), (1024, 24576, [256]), (1024, 24576, [777]), (1024, 4096, [140] * 16), (1024, 4096, [40] * 17),
             (512, 11009, [1500]), (512, 11009, [3000]), (256, 688, [1])]
    got = [any("stat_whole" in l["name"] for l in ls) for ls in launches.record([dict(entry="select", d=d, n=F, lens=v) for d, F, v in calls])]
    assert got == [True, False, True, False, True, False, True, False, True]


def test_statistic_in_chunks_where_one_kernel_would_leave_the_chip_idle():
    """Few columns: a workgroup has all rows of its columns, one load behind the other."""
    calls = [(64, 1000, [700], G.F32, True), (64, 1000, [1000], G.F32, False), (1024, 2623, [600], G.BF16, True), (1024, 2623, [2341], G.BF16, False),
             (184, 486, [2022], G.F32, False), (96, 287, [1779], G.F32, False), (64, 4096, [1000], G.BF16, True), (64, 4096, [1400], G.BF16, False),
             (64, 4096, [1400, 1400], G.BF16, False), (64, 4096, [1000] * 4, G.BF16, True), (64, 1400, [1400, 40, 40, 40], G.BF16, False),
             (64, 8192, [600], G.BF16, True), (64, 8192, [700], G.BF16, False), (64, 8193, [2000], G.BF16, True), (64, 11008, [1200], G.BF16, True),
             (64, 1400, [0, 1000], G.BF16, False), (64, 1400, [0, 0], G.BF16, True)]
    calls += [(d, F, lens, G.BF16, True) for d, F, lens in cases.LONG_WHOLE_CASES]
    got = [any("stat_whole" in l["name"] for l in ls) for ls in launches.record([dict(entry="select", d=d, n=F, lens=v, dtype=t) for d, F, v, t, _ in calls])]
    assert [(*c[:4], g) for c, g in zip(calls, got)] == calls


def test_fp32_outputs_take_sixteen_waves_where_that_is_faster():
    """Forms of the second product in fp32, with a top-k to carry and without: waves, sums of each, side of the tiles, a top-k apart."""
    calls = [("out", 256, 688, 250, G.F32), ("out", 256, 688, 500, G.F32), ("phase", 256, 688, 500, G.F32), ("out", 64, 128, 64, G.F32),
             ("phase", 64, 128, 64, G.F32), ("out", 512, 1400, 500, G.F32), ("out", 512, 2048, 500, G.F32), ("out", 1024, 4099, 77, G.F32),
             ("out", 512, 1001, 200, G.BF16), ("out", 512, 1004, 250, G.BF16), ("out", 96, 287, 1000, G.F32), ("phase", 96, 287, 1779, G.F32), ("out", 256, 688, 1500, G.F32)]
    got = []
    for (entry, d, F, S, _), ls in zip(calls, launches.record([dict(entry=e, d=d, n=F, lens=[S], dtype=dt) for e, d, F, S, dt in calls])):
        name = ls[-1]["name"]                # f32_out_topk_kernel: sixteen waves; f32_nt_kernel: eight, of one sum or two
        m = re.search(r"(?:f32_out_topk_kernelILb\dELb\dELi(\d)E|f32_nt_kernelILb0ELb0ELb\dELb\dELi(\d)ELi(\d)E)", name)
        got.append((entry, F, S, 16 if m[1] else 8, int(m[3] or 1), 16 * int(m[1] or m[2]), any("topk_reg" in l["name"] for l in ls)))
    assert got == [("out", 688, 250, 16, 1, 16, False), ("out", 688, 500, 8, 2, 32, False), ("phase", 688, 500, 16, 1, 32, False),
                   ("out", 128, 64, 8, 1, 32, False), ("phase", 128, 64, 16, 1, 16, False), ("out", 1400, 500, 8, 2, 32, False),
                   ("out", 2048, 500, 16, 1, 32, False), ("out", 4099, 77, 16, 1, 32, False), ("out", 1001, 200, 16, 1, 32, False),
                   ("out", 1004, 250, 8, 2, 32, False), ("out", 287, 1000, 8, 2, 32, False), ("phase", 287, 1779, 16, 1, 32, False),
                   ("out", 688, 1500, 8, 1, 32, False)]


def test_every_field_of_a_launch_is_set():
    """The row partials' stride of products that write none (raw ranges, outputs of a prompt) and of those that do."""
    calls = [dict(entry="select", d=2560, n=17424, lens=[47]), dict(entry="out", d=512, n=4096, lens=[40]),
             dict(entry="select", d=512, n=1000, lens=[300])]
    got = [[l for l in ls if launches.form(l["name"])][0] for ls in launches.record(calls)]
    assert [" raw " in launches.form(l["name"]) for l in got] == [True, True, False]
    assert [l["nt_row"] for l in got] == [0, 0, got[2]["nt"]]


def test_columns_of_tiles_begin_at_other_k_tiles_by_the_bytes_that_are_read():
    """Not by the rows' stride: interleaved and padded rows read no more than d of it."""
    calls = [(dict(entry="select", d=4096, n=9800, lens=[64]), 1), (dict(entry="select", d=4096, n=8600, lens=[40]), 0),
             (dict(entry="select", d=4096, n=5504, lens=[40], ld=3 * 4096), 0), (dict(entry="select", d=4096, n=7168, lens=[100], ld=3 * 4096), 0),
             (dict(entry="select", d=4096, n=8750, lens=[64], ld=3 * 4096), 1), (dict(entry="select", d=4096, n=7168, lens=[100], ld=8192), 0),
             (dict(entry="select", d=5120, n=6912, lens=[100], ld=8192), 1), (dict(entry="select", d=5120, n=13824, lens=[40]), 0),
             (dict(entry="select", d=4096, n=20000, lens=[100], gated=False), 1), (dict(entry="select", d=4096, n=13000, lens=[40], gated=False, ld=8192), 0),
             (dict(entry="select", d=4096, n=11008, lens=[260]), 0), (dict(entry="out", d=6144, n=12288, lens=[40]), 1),
             (dict(entry="out", d=4096, n=12288, lens=[40], ldw=4 * 12288), 0)]
    first = [[l for l in ls if launches.form(l["name"])][0] for ls in launches.record([c for c, _ in calls])]
    assert [(c, l["rotate"]) for (c, _), l in zip(calls, first)] == calls
