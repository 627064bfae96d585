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
