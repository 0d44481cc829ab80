"""Which form of the prompt product a call takes, and what it makes of it (no GPU: tests/launches.py)."""
import launches


def routes(calls):
    return [[launches.route(l) for l in ls if launches.form(l["name"])] for ls in launches.record(calls)]


# d, D_ff, tokens of an Eq. 3 block whose products are summed in parts; the form, and sums kept apart in registers (1: ranges with slabs)
PARTS = [
    (4096, 11008, 40, "64x64 Eq. 3 copy", 4),
    (4608, 21712, 316, "128x128 Eq. 3", 2),
    (8128, 12304, 108, "128x64 Eq. 3 copy", 5),
    (3648, 9488, 196, "224x128 raw Eq. 3", 1),        # 256 x 64 tiles would wait
    (2048, 8912, 237, "256x128 raw Eq. 3", 1),
    (6144, 16288, 100, "128x128 raw Eq. 3", 1),       # 128 x 64 tiles would
    (2816, 18128, 24, "64x128 raw Eq. 3", 1),         # 128 x 128 tiles of which 24 tokens are there
    (2560, 24768, 1, "64x128 raw Eq. 3", 1),
    (1600, 2992, 14, "64x128 raw Eq. 3", 1),          # 47 tiles of 64 x 64
]


def test_sums_stay_apart_in_registers_only_where_that_is_faster():
    got = routes([dict(entry="select", d=d, n=F, lens=[S]) for d, F, S, *_ in PARTS])
    assert [(*c[:3], r[0][0], r[0][3]) for c, r in zip(PARTS, got)] == PARTS
