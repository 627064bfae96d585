"""Launch grid of the finetune unit's weight GEMM (host logic, no GPU): with the workgroup-to-tile rules its header
states every tile of the output, or every range of K of a tile that is cut, is computed exactly once, the workgroups an XCD
runs together cover a compact block of tiles, the ranges of K follow the device alone, and the tile height follows the share
of its compute units a stream may use (Harli Sec. 6.2: the finetune task runs on a share of them)."""
import itertools

import pytest

from paper_2511_11729_amd import binding as hb


def tiles_of(plan, M, tiles_n, tile_rows):
    GM, GN, total, chunk = plan["GM"], plan["GN"], plan["total"], plan["chunk"]
    nbn = -(-tiles_n // GN)
    cover = {}
    for w in range(plan["grid"]):
        slot = (w & 7) * chunk + (w >> 3)
        if slot >= total:
            continue
        blk, within = divmod(slot, GM * GN)
        bm, bn = divmod(blk, nbn)
        tm, tn = bm * GM + within // GN, bn * GN + within % GN
        if tm * tile_rows >= M or tn >= tiles_n:
            continue
        cover.setdefault((tm, tn), []).append(w)
    return cover


SHAPES = [(2048, 16), (2048, 48), (2048, 86), (2048, 43), (300, 3), (129, 1), (4096, 172), (1000, 7), (64, 5)]


@pytest.mark.parametrize("M,tiles_n", SHAPES)
@pytest.mark.parametrize("tile_rows", [128, 256])
@pytest.mark.parametrize("n_cu", [256, 230, 179, 7])
def test_every_tile_is_computed_once(M, tiles_n, tile_rows, n_cu):
    p = hb.dbg_gemm2_plan(M, tiles_n, tile_rows, n_cu)
    tiles_m = -(-M // tile_rows)
    cover = tiles_of(p, M, tiles_n, tile_rows)
    assert set(cover) == set(itertools.product(range(tiles_m), range(tiles_n)))
    assert all(len(ws) == 1 for ws in cover.values())
    assert p["grid"] == p["chunk"] * 8 and p["rounds"] == -(-tiles_m * tiles_n // n_cu)
    # the 32 workgroups an XCD runs at a time (consecutive slots of its chunk) stay inside one or two blocks of tiles
    if p["total"] >= 8 * 32 and p["GM"] * p["GN"] == 32:
        for x in range(8):
            first = [(x * p["chunk"] + i) // 32 for i in range(32)]
            assert len(set(first)) <= 2


def test_bad_arguments():
    with pytest.raises(hb.HarliError):
        hb.dbg_gemm2_plan(2048, 16, 100, 230)
    with pytest.raises(hb.HarliError):
        hb.dbg_gemm2_plan(2048, 16, 128, 0)


@pytest.mark.parametrize("M,tiles_n,stages", [(2048, 16, 129), (2048, 48, 129), (4096, 20, 434), (48, 16, 345), (600, 20, 434), (129, 5, 40)])
@pytest.mark.parametrize("share", [230, 128, 26])
def test_a_share_of_the_compute_units_moves_the_tile_height_and_no_range_of_k(M, tiles_n, stages, share):
    """The ranges of K decide the order of the sums: those of a confined stream are the device's, over the same tiles."""
    whole, part = hb.dbg_gemm2_cut(M, tiles_n, stages, 256), hb.dbg_gemm2_cut(M, tiles_n, stages, 256, share)
    assert part["ks"] == whole["ks"] and (part["full"] == 0) == (whole["full"] == 0)
    if whole["full"] and whole["rest"]:
        assert part == whole                                  # which tiles are cut depends on the tile height
    assert M > 128 or part["rows"] == 128


def test_tile_height_on_nine_tenths_of_the_chip():
    """2048 x 4096 x 4096 is one round of 128-row tiles on 256 compute units, and on 230 one of 256-row tiles."""
    assert hb.dbg_gemm2_cut(2048, 16, 128, 256)["rows"] == 128
    part = hb.dbg_gemm2_cut(2048, 16, 128, 256, 230)
    assert part["rows"] == 256 and part["ks"] == 1 and part["full"] == 128


def test_passes_of_a_small_workspace_cover_the_cut_tiles():
    """The plan knows no workspace; with less of it than the partial tiles take, equal passes of whole tiles."""
    full = hb.dbg_gemm2_cut(600, 20, 434, 256)
    tile = full["ks"] * full["rows"] * 256 * 4
    assert full["ks"] > 2 and full["per_pass"] == full["rest"]
    for fit in (full["rest"], full["rest"] - 1, 7, 1, 0):
        c = hb.dbg_gemm2_cut(600, 20, 434, 256, part_bytes=fit * tile + tile // 2)
        assert {k: v for k, v in c.items() if k != "per_pass"} == {k: v for k, v in full.items() if k != "per_pass"}
        assert c["per_pass"] <= fit and (c["per_pass"] > 0) == (fit > 0)
        assert fit == 0 or -(-c["rest"] // c["per_pass"]) == -(-c["rest"] // fit)   # no more passes than it takes
    for M, tiles_n, stages in ((4096, 200, 2000), (48, 16, 690), (300, 1, 64)):       # the library's smallest workspace: 4 MiB
        c = hb.dbg_gemm2_cut(M, tiles_n, stages, 256, part_bytes=4 << 20)
        assert c["ks"] == 1 or c["per_pass"] >= 1


@pytest.mark.parametrize("M,tiles_n,stages", [(1032, 14, 1186), (1100, 5, 40), (48, 16, 345), (2048, 48, 129), (1032, 74, 112), (4096, 20, 434),
                                              (300, 1, 64), (2304, 3, 17), (129, 172, 33)])
@pytest.mark.parametrize("n_cu,share", [(256, 256), (256, 230), (256, 26), (7, 7)])
@pytest.mark.parametrize("part_bytes", [4 << 20, 64 << 20])
def test_every_range_of_every_tile_is_computed_once(M, tiles_n, stages, n_cu, share, part_bytes):
    """Cut launches, pass by pass: whole tiles, ranges of the others, several bands of row tiles with a ragged last one."""
    c = hb.dbg_gemm2_cut(M, tiles_n, stages, n_cu, share, part_bytes)
    assert c["tiles_m"] == -(-M // c["rows"]) and c["full"] + c["rest"] == c["tiles_m"] * c["tiles_n"]
    if c["ks"] == 1:
        assert c["rest"] == 0
        return

    def place(t):
        band, rem = divmod(t, c["GM"] * c["tiles_n"])
        rows = min(c["GM"], c["tiles_m"] - band * c["GM"])
        return band * c["GM"] + rem % rows, rem // rows
    done, first, full = {}, c["full"], c["full"]
    while first < c["full"] + c["rest"]:
        rest = min(c["per_pass"], c["full"] + c["rest"] - first)
        assert rest * c["ks"] * c["rows"] * 256 * 4 <= part_bytes
        chunk_full, chunk_cut = -(-full // 8), -(-rest * c["ks"] // 8)
        if rest == c["rest"]:
            assert (chunk_full, chunk_cut) == (c["chunk_full"], c["chunk_cut"])
        for w in range(8 * chunk_full):
            slot = (w & 7) * chunk_full + (w >> 3)
            if slot < full:
                done.setdefault(place(slot), []).append("whole")
        for w in range(8 * chunk_cut):
            piece = (w & 7) * chunk_cut + (w >> 3)
            if piece < rest * c["ks"]:
                done.setdefault(place(first + piece % rest), []).append(piece // rest)
        first, full = first + rest, 0
    assert set(done) == set(itertools.product(range(c["tiles_m"]), range(c["tiles_n"])))
    assert all(v == ["whole"] or sorted(v) == list(range(c["ks"])) for v in done.values())


# ---- every launch in the order it runs in, by operand and output type -------------------------------------------------
def tile_of(c, t):
    band, rem = divmod(t, c["GM"] * c["tiles_n"])
    rows = min(c["GM"], c["tiles_m"] - band * c["GM"])
    return band * c["GM"] + rem % rows, rem // rows


@pytest.mark.parametrize("half,f32out", [(True, False), (True, True), (False, False), (False, True)])
@pytest.mark.parametrize("share", [256, 230, 26])
def test_every_tile_of_an_uncut_launch_is_computed_once(half, f32out, share):
    """Both orders: blocks where whole ones cover the matrix, else bands without an empty slot; every tile height."""
    seen = set()
    for M, tiles_n, stages in itertools.product((1, 130, 160, 300, 600, 1032, 1100, 2048, 2304, 3000, 3400, 4096), (1, 5, 16, 43, 48, 86, 100), (3, 33, 129)):
        c = hb.dbg_gemm2_cut(M, tiles_n, stages, 256, share, half=half, f32out=f32out)
        assert c["tiles_m"] == -(-M // c["rows"]) and c["full"] + c["rest"] == c["tiles_m"] * tiles_n
        p = hb.dbg_gemm2_plan(M, tiles_n, c["rows"], 256)
        whole_blocks = p["total"] == c["tiles_m"] * tiles_n
        assert c["banded"] == (c["ks"] > 1 or not whole_blocks)
        if c["ks"] > 1:
            continue
        seen.add((c["rows"], c["banded"]))
        if c["banded"]:
            assert c["rest"] == 0 and c["full"] == c["tiles_m"] * tiles_n and c["chunk_full"] == -(-c["full"] // 8)
            slots = [(w & 7) * c["chunk_full"] + (w >> 3) for w in range(8 * c["chunk_full"])]
            done = [tile_of(c, s) for s in slots if s < c["full"]]
        else:
            cover = tiles_of(p, M, tiles_n, c["rows"])
            done = [t for t, ws in cover.items() for _ in ws]
        assert sorted(done) == list(itertools.product(range(c["tiles_m"]), range(tiles_n)))
    heights = {128, 160, 192, 224, 256} if half and share == 256 else {128, 256}
    assert {rows for rows, _ in seen} >= heights and {b for _, b in seen} == {0, 1}


@pytest.mark.parametrize("tile_rows", [160, 192, 224])
@pytest.mark.parametrize("M,tiles_n", SHAPES + [(2240, 16), (3840, 40)])
def test_the_block_order_of_the_other_heights(tile_rows, M, tiles_n):
    p = hb.dbg_gemm2_plan(M, tiles_n, tile_rows, 256)
    cover = tiles_of(p, M, tiles_n, tile_rows)
    assert set(cover) == set(itertools.product(range(-(-M // tile_rows)), range(tiles_n)))
    assert all(len(ws) == 1 for ws in cover.values()) and p["grid"] == p["chunk"] * 8


@pytest.mark.parametrize("half", [True, False])
@pytest.mark.parametrize("share", [256, 230, 26])
def test_every_range_of_every_tile_with_fp32_outputs_or_bfloat16_operands(half, share):
    """As above for cut launches; passes of a small workspace."""
    cut = 0
    for (M, tiles_n, stages), part_bytes in itertools.product(((2048, 16, 129), (1032, 14, 1186), (600, 20, 434), (300, 1, 64), (4096, 20, 434),
                                                               (1100, 5, 40), (2304, 3, 17)), (4 << 20, 64 << 20)):
        c = hb.dbg_gemm2_cut(M, tiles_n, stages, 256, share, part_bytes, half=half, f32out=True)
        assert c["tiles_m"] == -(-M // c["rows"]) and c["full"] + c["rest"] == c["tiles_m"] * tiles_n
        assert half or c["rows"] in (128, 256)
        if c["ks"] == 1:
            continue
        cut += 1
        done, first, full = [], c["full"], c["full"]
        while first < c["full"] + c["rest"]:
            rest = min(c["per_pass"], c["full"] + c["rest"] - first)
            assert rest > 0 and rest * c["ks"] * c["rows"] * 256 * 4 <= part_bytes
            chunk_full, chunk_cut = -(-full // 8), -(-rest * c["ks"] // 8)
            done += [(tile_of(c, s), "whole") for s in ((w & 7) * chunk_full + (w >> 3) for w in range(8 * chunk_full)) if s < full]
            done += [(tile_of(c, first + q % rest), q // rest) for q in ((w & 7) * chunk_cut + (w >> 3) for w in range(8 * chunk_cut)) if q < rest * c["ks"]]
            first, full = first + rest, 0
        want = [(tile_of(c, t), "whole") for t in range(c["full"])] + [(tile_of(c, t), r) for t in range(c["full"], c["full"] + c["rest"]) for r in range(c["ks"])]
        assert sorted(done, key=str) == sorted(want, key=str) and len({tile_of(c, t) for t in range(c["tiles_m"] * tiles_n)}) == c["tiles_m"] * tiles_n
    assert cut >= 6


def test_the_output_type_moves_the_plan():
    """A store of fp32 with its residual costs more than one of 16 bits: 2048 x 4096 over 129 stages goes out whole in 128 rows
    as half, and in two ranges of 256 rows as fp32 (the o projection of the 7B shape)."""
    a, b = hb.dbg_gemm2_cut(2048, 16, 129, 256), hb.dbg_gemm2_cut(2048, 16, 129, 256, f32out=True)
    assert (a["rows"], a["ks"]) == (128, 1) and (b["rows"], b["ks"]) == (256, 2)
