"""The rules that give a matrix phase its kernel, tiles and reduction parts (csrc/rows_plan.h), compiled for the CPU."""
import os
import subprocess

import pytest

from plan_cases import BODY_TILES, HEAD_TILES, LIST_GROUPS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256
PART_FLOATS = 16384 * 4 * 256  # the smallest room for partial sums a workspace has
ALL_FEW, FEW, TILES, CORE = -1, 0, 1, 2  # the kernel of a phase (ALL_FEW: of every phase of the call)


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "rows_plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(ROOT, "tests", "plan", "rows_plan_driver.cpp"),
                    "-o", exe], check=True)
    return exe


@pytest.fixture(scope="module")
def plan(driver):
    exe = driver

    def ask(calls):
        # (call_rows: rows of the whole call, of which `rows` share an id list; d: the head's width)
        lines = "\n".join("%d %d %d %d %d %d %d %d %d" % (c["K"], -(-c["n"] // 16) * 16, c["rows"], c.get("head", 0),
                                                             c.get("pairs", 0), CUS, PART_FLOATS,
                                                             c.get("call_rows", c["rows"]), c.get("d", c["K"]))
                          for c in calls)
        out = subprocess.run([exe], input=lines, capture_output=True, text=True, check=True).stdout.split("\n")
        keys = ("route", "bm", "bn", "parts", "us")
        return [dict(zip(keys, map(float, l.split()))) for l in out if l]

    return ask


@pytest.mark.parametrize("rows", [2, 5, 16, 17, 33, 64])
@pytest.mark.parametrize("K", [288, 544, 1056, 2080, 4128, 8160])
@pytest.mark.parametrize("n", [1024, 4096, 32768])
def test_a_reduction_of_an_odd_number_of_32s_gets_the_tiles_of_its_neighbours(plan, rows, K, n):
    """Model widths are multiples of 32; the tiles for few rows walk a reduction in steps of 64, the last of them half a step.
    Such a call is estimated, and cut, like the next whole number of steps."""
    odd, even = plan([dict(K=K, n=n, rows=rows), dict(K=K + 32, n=n, rows=rows)])
    assert odd["bm"] <= max(16, 2 * rows)
    assert odd["us"] <= even["us"] * 1.001


HEADS = [1024, 4096, 8195, 16384, 24576, 29500, 30336, 32768, 32769, 33000, 36000, 40000, 49152, 65536, 65537, 75841,
         98304, 118000, 131072, 151680, 262144, 400000]


@pytest.mark.parametrize("rows,call_rows", [(2, 2), (5, 5), (16, 16), (2, 40), (5, 40), (16, 40)])
@pytest.mark.parametrize("K", [256, 512, 544, 1024, 1056, 2048, 2080, 3072, 4096, 4128, 5120, 8192])
def test_few_rows_take_the_tiles_only_where_their_rounds_are_full(plan, rows, call_rows, K):
    """Up to 16 rows, by themselves or sharing a list in a larger batch, few_rows.h is the alternative.  The tiled product is taken
    in one round of workgroups and where further rounds are nearly full, never in tiles of many times the rows: a head of
    151680 x 2048 in 593 blocks for 256 units was 23 us slower per step, one of 75841 x 3072 in tiles of 128 rows 18 us."""
    tiles = 0
    for n, p in zip(HEADS, plan([dict(K=K, n=n, rows=rows, head=1, call_rows=call_rows) for n in HEADS])):
        assert p["route"] != CORE
        assert (p["route"] == ALL_FEW) == (call_rows <= 16 and (K >= 384 if rows <= 8 else K > 2048))
        if p["route"] != TILES:
            continue
        tiles += 1
        blocks = -(-n // p["bn"])
        assert p["us"] < 1e29 and blocks >= 1 and p["parts"] >= 1  # there is a plan
        assert p["bm"] <= 64, (n, p)
        assert p["parts"] > 1 or blocks <= 1024
        slots = -(-blocks // CUS) * CUS
        assert blocks <= CUS or (K <= 2048 and K % 64 == 0 and blocks >= 0.9 * slots), (n, p)
        if K > 2048 and n * K * 2 > 32e6:  # large heads: a nearly full round, in whichever tile
            assert blocks > 0.9 * slots - 1 or (p["bn"] == 256 and blocks > 0.5 * slots), (n, p)
    assert tiles or call_rows <= 16


@pytest.mark.parametrize("rows,K,n,expect", [
    (16, 4096, 32768, 16), (16, 4096, 30336, 16), (16, 4096, 33000, 64), (5, 4096, 40000, 64), (2, 4096, 65536, 64),
    (16, 4096, 131072, 0), (16, 4096, 75841, 0), (16, 4096, 98304, 0), (2, 4096, 151680, 0), (16, 3072, 75841, 0),
    (5, 1024, 75841, 0), (5, 1024, 151680, 0), (5, 512, 75841, 0), (16, 2048, 36000, 64), (5, 1056, 65536, 0),
    (16, 2048, 131072, 64), (8, 2048, 98304, 0), (8, 2016, 32768, 16), (8, 2016, 33000, 0), (16, 3072, 24576, 0)])
def test_route_of_heads_at_few_rows(plan, rows, K, n, expect):
    """Rows that share a list in a larger batch: the tile's rows, or 0 for few_rows.h, on both sides of the lines."""
    p = plan([dict(K=K, n=n, rows=rows, head=1, call_rows=40)])[0]
    assert (p["bm"] if p["route"] == TILES else FEW) == expect, p


@pytest.mark.parametrize("rows,d,K,n,head,expect", [
    (2, 256, 256, 1024, 1, TILES), (8, 352, 352, 32768, 1, TILES), (8, 352, 704, 352, 0, TILES), (8, 352, 968, 352, 0, FEW),
    (8, 256, 256, 524309, 1, FEW), (2, 384, 384, 1024, 1, ALL_FEW), (8, 2048, 2048, 32768, 1, ALL_FEW),
    (9, 384, 384, 1024, 1, TILES), (9, 2048, 2048, 32768, 1, TILES), (9, 2048, 2048, 75841, 1, FEW), (9, 2048, 5640, 2048, 0, FEW),
    (9, 2080, 2080, 2111, 1, ALL_FEW), (16, 4096, 4096, 32768, 1, ALL_FEW), (17, 4096, 4096, 32768, 1, TILES),
    (17, 4096, 11000, 4096, 0, CORE), (17, 256, 256, 524309, 1, CORE)])
def test_kernel_of_a_phase(plan, rows, d, K, n, head, expect):
    """Both sides of every line between the kernels of several rows."""
    assert plan([dict(K=K, n=n, rows=rows, head=head, d=d)])[0]["route"] == expect


@pytest.mark.parametrize("d,rows,n", [(d, rows, n) for d, groups in LIST_GROUPS for rows, n in groups])
def test_lists_that_run_on_the_gpu_in_row_major_order(plan, d, rows, n):
    """test_gpu_parity.py runs these lists of a larger batch through few_rows.h."""
    call_rows = sum(r for r, _ in dict(LIST_GROUPS)[d])
    p = plan([dict(K=d, n=n, rows=rows, head=1, call_rows=call_rows)])[0]
    assert p["route"] == FEW and call_rows > 16, p


@pytest.mark.parametrize("d,vocab,rows,tile", HEAD_TILES)
def test_tiles_of_the_output_heads_that_run_on_the_gpu(plan, d, vocab, rows, tile):
    """Changed constants do not silently drop a tile, or the split head, from test_gpu_parity.py."""
    p = plan([dict(K=d, n=vocab, rows=rows, head=1)])[0]
    assert p["route"] == TILES and (p["bm"], p["bn"], p["parts"] > 1) == tile, p


@pytest.mark.parametrize("d,d_ffn,rows,tiles", BODY_TILES)
def test_tiles_of_the_body_phases_that_run_on_the_gpu(plan, d, d_ffn, rows, tiles):
    got = plan([dict(c, rows=rows, d=d) for c in (dict(K=2 * d, n=d), dict(K=d, n=2 * d_ffn, pairs=1), dict(K=d_ffn, n=d))])
    assert all(p["route"] == TILES for p in got)
    assert tuple((p["bm"], p["bn"], p["parts"] > 1) for p in got) == tiles, got


def test_every_tile_has_a_gpu_test():
    """Each tile, the small ones with the whole reduction and with a part of it."""
    ran = {t for *_, t in HEAD_TILES} | {t for *_, ts in BODY_TILES for t in ts}
    assert {t[:2] for t in ran} == {(256, 256), (128, 512), (128, 384), (64, 256), (64, 128), (32, 128), (16, 128)}
    assert {(bm, 128, split) for bm in (16, 32, 64) for split in (False, True)} <= ran
    # in parts, with a half step in the last: a width or d_ffn that is 32 modulo 64
    halves = {t for d, _, _, t in HEAD_TILES if d % 64} | {ts[2] for _, f, _, ts in BODY_TILES if f % 64}
    assert {(bm, 128, True) for bm in (16, 32, 64)} <= halves


# d_model, query heads, KV heads, head dimension, d_ffn, rows of the output head, capacity: three steps of one sequence were slower
# on a quarter of the units than with a launch per phase (False), or faster (True)
NARROW = [
    (256, 4, 2, 64, 688, 1024, 192, True), (256, 4, 2, 64, 688, 4096, 16384, True), (256, 4, 4, 64, 688, 4096, 1024, True),
    (256, 4, 2, 64, 688, 6144, 1024, True), (384, 3, 3, 128, 1024, 1024, 384, True),
    (256, 4, 4, 64, 688, 8192, 128, True), (320, 5, 5, 64, 864, 4096, 1024, True), (480, 8, 2, 64, 1280, 3072, 192, False),
    (256, 16, 4, 64, 688, 1024, 32832, False), (256, 16, 4, 64, 688, 4096, 16448, False),
    (256, 16, 16, 64, 688, 1024, 16448, False), (320, 5, 5, 64, 864, 1024, 32832, False),
    (256, 4, 2, 64, 688, 12288, 1024, True), (256, 16, 4, 64, 688, 4096, 8256, True), (256, 4, 2, 64, 688, 16384, 192, False),
    (480, 8, 2, 64, 1280, 14336, 1024, False),  # (slower or about equal; 480 wide meets at 18.7 MiB, the line is that of 256)
]


@pytest.mark.parametrize("d,hq,hkv,hd,d_ffn,n,cap,single", NARROW)
def test_narrow_heads_take_the_single_launch_where_it_is_ahead(driver, d, hq, hkv, hd, d_ffn, n, cap, single):
    """The rule against both sides' times: by the weights of a step and the keys and values that a context can grow to."""
    step = 2 * (d * (2 * d + (hq + 2 * hkv) * hd + hq * hd + 3 * d_ffn) + n * d)
    out = subprocess.run([driver, "narrow"], input=f"{step} {4 * hkv * hd * cap}", capture_output=True, text=True, check=True)
    assert out.stdout.split() == [str(int(single))], (step, 4 * hkv * hd * cap)


@pytest.mark.parametrize("positions,sequences,groups,sized,cap,small", [
    (1, 512, 1024, 0, 512, 0),                                                       # one position: never
    (509, 1, 1024, 0, 512, 1), (2, 4, 8, 1, 2048, 1), (64, 8, 512, 0, 1088, 1),      # up to 16 rounds of 128 tokens: always
    (4, 16, 128, 1, 2049, 0), (4, 16, 128, 1, 4160, 0), (4, 16, 128, 1, 32832, 0),   # more, and splits by the lengths that are there
    (8, 64, 512, 0, 4160, 1), (8, 64, 512, 0, 5120, 1), (8, 64, 512, 0, 5121, 0),    # more, and contexts that may differ
    (8, 64, 1024, 0, 32832, 0), (4, 8, 32, 0, 4160, 0),
    (500, 1, 1000, 0, 32832, 1), (64, 1, 128, 1, 8256, 0), (64, 1, 130, 1, 8256, 1), # one sequence
])
def test_attention_of_a_block_by_rounds_and_groups(driver, positions, sequences, groups, sized, cap, small):
    """Small workgroups where no context can be long enough to keep the chip waiting for one wave's rounds; never in a block whose
    splits the vector attention serves."""
    out = subprocess.run([driver, "block"], input="".join(f"{positions} {mc} {sequences} {groups} {sized} {cap}\n" for mc in (1, 0)),
                         capture_output=True, text=True, check=True)
    assert out.stdout.split() == [str(small), "0"]
