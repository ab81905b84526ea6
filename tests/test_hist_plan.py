"""Host-side checks of the histogram launch plans (no GPU): the index arithmetic of the histogram kernels, of the
hand-over of a row group's local bins to its slot and of the slot reduction is replayed in numpy from the plan the
library reports for a shape (qgbdt_describe_hist_plan), and every address is checked against the sizes of what it
points into -- the matrix, the local bins, the workspace section of the slots, the histogram."""
import itertools

import numpy as np
import pytest

from paper_2207_09682_amd.binding import describe_counting, describe_hist_plan, describe_row_group, describe_segment_order

SHAPES = [  # n_rows, n_features, n_bins, max_leaves, bin_bytes
    (10_500_000, 28, 255, 255, 1), (1_000_000, 28, 255, 255, 1), (10_000, 28, 63, 15, 1),
    (400_000, 2000, 63, 63, 1), (20_000_000, 200, 255, 511, 1), (463_715, 90, 255, 255, 1),
    (5000, 3, 256, 15, 1), (9000, 5, 16, 15, 1), (5000, 65, 255, 31, 1), (7000, 64, 256, 31, 1),
    (5000, 36, 100, 31, 1), (30_000, 72, 256, 31, 1), (100_000, 1, 2, 4, 1), (100_000, 2048, 256, 15, 1),
    (20_000, 10, 600, 31, 2), (9000, 33, 1024, 31, 2), (5000, 100, 300, 31, 2), (3000, 1, 700, 7, 2),
    (2_000_000, 40, 600, 63, 2), (160_000_000, 28, 255, 15, 1), (2_400_000, 2000, 63, 7, 1),
    # edges: very wide rows, many bins of both widths, tile widths around the 128-byte piece, the leaf limit
    (50_000, 4096, 256, 31, 1), (20_000, 10_000, 64, 15, 1), (3000, 2000, 1024, 7, 2), (1000, 7, 2, 658, 1),
    (300, 255, 256, 7, 1), (100_000, 16, 256, 15, 1), (100_000, 124, 255, 15, 1), (100_000, 128, 255, 15, 1),
    (50_000, 132, 200, 15, 1), (8000, 257, 1024, 15, 2),
    # long narrow matrices of other row widths (two-level byte-stream builds)
    (3_000_000, 16, 255, 15, 1), (3_000_000, 40, 255, 15, 1), (3_000_000, 48, 255, 15, 1), (6_000_000, 20, 100, 15, 1),
]
BITS = [(2, 2), (3, 3), (4, 4), (5, 5), (3, 8), (3, 0), (8, 8)]


def _plans(shape):
    N, F, nb, L, bb = shape
    for (bg, bh), acc, skew in itertools.product(BITS, (0, 16, 32), (False, True)):
        yield (bg, bh, acc, skew), describe_hist_plan(N, F, nb, L, bb, bg, bh, acc, skew)


def _rows_fitting_word32(bg, bh, s):
    kg, kh = 2 ** (bg - 1) - 1, (2 ** bh - 2 if bh else 1)
    return min((2 ** (31 - s) - 1) // kg, (2 ** s - 1) // kh)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}_nb{s[2]}_L{s[3]}_b{s[4]}")
def test_plan_invariants(shape):
    N, F, nb, L, bb = shape
    for key, p in _plans(shape):
        bg, bh, acc, skew = key
        wbytes = 4 if p["acc_width"] == 16 else 8
        npd = 4 // bb
        # tiles cover the features, local bins fit the LDS, and only the wide-row kernels go beyond 64 KB
        assert p["n_tiles"] == -(-F // p["ft"]) and p["ft"] >= 1
        assert p["lds_bytes"] <= 160 * 1024
        assert p["lds_bytes"] <= 64 * 1024 or p["wide_v"] > 0, key
        assert p["slot_bytes"] >= p["lds_bytes"] and p["slot_bytes"] % 16 == 0
        # the flat grid is cut into (XCD, tile, lane): lanes come in whole groups of 8
        assert p["max_lanes"] % 8 == 0 and p["max_lanes"] >= 8 and p["max_groups"] >= 1
        # the slots of any launch of this shape lie inside the workspace section sized from the shape alone
        assert p["max_items"] * p["n_tiles"] * p["slot_bytes"] <= p["partial_bytes"], key
        # width rule (Sec. 7.4.3): a chunk never holds more rows than the fields of a local word take
        if p["acc_width"] == 16:
            assert p["chunk_rows"] <= _rows_fitting_word32(bg, bh, p["hshift"]), key
            assert p["chunk_rows"] >= max(_rows_fitting_word32(bg, bh, s) for s in range(8, 25)), key   # the best split
        assert 1 <= p["single_rows"] <= p["chunk_rows"]
        last = F - (p["n_tiles"] - 1) * p["ft"]
        if not p["bytewise"]:
            assert p["dpr"] * p["rows_per_it"] <= 64 and p["rows_per_it"] >= 1
            assert last >= min(npd, F), key                          # every tile row holds a whole dword
            if p["wide_v"]:
                assert bb == 1 and F % p["wide_v"] == 0 and p["ft"] % p["wide_v"] == 0 and last % p["wide_v"] == 0
                assert p["ftp"] == (p["ft"] + p["ft"] // 4 if p["pad16"] else p["ft"])
            else:
                assert p["ftp"] >= p["ft"]
            assert p["lds_bytes"] == p["ftp"] * nb * wbytes
        if p["flat_lanes"]:
            assert bb == 1 and p["n_tiles"] == 1 and (16 * p["flat_lanes"]) % F == 0 and p["flat_lanes"] <= 64
            assert p["flat_rows"] * F == 16 * p["flat_lanes"]


def _walk_two_level_groups(p, F, count, begin, groups):
    """The two-level byte-stream kernel's walk over one build of `count` rows from row `begin`: every row lies in
    exactly one group, whole blocks start 16-byte aligned, and no more rows than a chunk holds are added to the 32-bit
    working words between two folds."""
    n_waves, U = 16, 2
    align_rows = 16 // (16 if F % 16 == 0 else 8 if F % 8 == 0 else 4)
    BR = U * p["flat_rows"]
    head = min(count, (align_rows - begin % align_rows) % align_rows)
    rpg = max(BR, -(-(-(-(count - head) // groups)) // BR) * BR)
    fold_rounds = max(1, (p["chunk_rows"] - BR - align_rows) // (n_waves * BR))
    covered = head
    for g in range(groups):
        gbegin = min(count, head + g * rpg)
        gend = min(count, gbegin + rpg)
        grow = gend - gbegin
        n_blocks = grow // BR
        rounds = -(-n_blocks // n_waves)
        if n_blocks:
            assert ((begin + gbegin) * F) % 16 == 0
        since_fold = 0
        for r in range(rounds):
            since_fold += BR * max(0, min(n_waves, n_blocks - r * n_waves))
            if (r + 1) % fold_rounds == 0 and r + 1 < rounds:
                assert since_fold <= p["chunk_rows"]
                since_fold = 0
        since_fold += (grow - n_blocks * BR) + (head if g == 0 else 0)
        assert since_fold <= p["chunk_rows"], (F, count, begin, g)
        assert (begin + gend) * F <= (begin + count) * F                             # the last load ends inside the slice
        covered += grow
    assert covered == count


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}_nb{s[2]}_L{s[3]}_b{s[4]}")
def test_plan_of_one_long_contiguous_build(shape):
    # the plan of a stand-alone build of all rows: for narrow matrices the byte-stream kernel's two-level form
    # (32-bit working words folded into 64-bit words in LDS), whose slots hold the 64-bit words
    N, F, nb, L, bb = shape
    seen_two = False
    for (bg, bh), acc in itertools.product(BITS, (0, 16, 32)):
        p = describe_hist_plan(N, F, nb, L, bb, bg, bh, acc, False, rows=N, n_builds=1)
        assert p["max_items"] * p["n_tiles"] * p["slot_bytes"] <= p["partial_bytes"]
        assert p["max_lanes"] % 8 == 0 and p["lds_bytes"] <= 160 * 1024
        groups = -(-N // p["target_rows"])
        assert 1 <= groups <= p["max_items"]
        if p["two_level"]:
            seen_two = True
            words = nb * p["ftp"]
            assert acc != 32 and p["acc_width"] == 16 and p["flat_lanes"] > 0 and p["n_tiles"] == 1 and p["threads"] == 1024
            assert p["lds_bytes"] == ((4 * words + 15) // 16) * 16 + 8 * words
            assert p["slot_bytes"] >= 8 * words and p["slot_bytes"] % 16 == 0
            assert groups <= p["max_lanes"] == 256                                   # one group per CU, all resident
            assert p["chunk_rows"] <= _rows_fitting_word32(bg, bh, p["hshift"])      # the working words still follow the width rule
            assert N >= 2 * 256 * p["chunk_rows"]
            for begin in (0, 1, 3):                                                  # a slice that starts off a 16-byte boundary
                _walk_two_level_groups(p, F, N - begin, begin, -(-(N - begin) // p["target_rows"]))
        else:
            # without the fold a group of 32-bit words must not be longer than the item table allows one-chunk groups, or the width is 64
            assert p["acc_width"] == 32 or acc == 16 or N // p["single_rows"] < p["max_items"] - 2
    if bb == 1 and 16 <= F <= 64 and F % 4 == 0 and N >= 2_000_000:
        assert seen_two


def _lane_columns(p, F, bb, tile, dword_kernel=False):
    """(first byte of the lane's load inside the row, bytes loaded, LDS word columns it may update) per active lane of
    one tile, as the dword-per-lane and the wide-row kernels compute them."""
    npd = 4 // bb
    f0 = tile * p["ft"]
    ft = min(p["ft"], F - f0)
    out = []
    if p["wide_v"] and not dword_kernel:
        V = p["wide_v"]
        P = p["ft"] // V
        for lane in range(64):
            c = lane % P
            if V * c >= ft:
                continue                                             # the lane sits out (its load aliases piece 0)
            cols = [20 * c + 4 * i + k for i in range(4) for k in range(4)] if V == 16 else [8 * c + k for k in range(8)]
            out.append((f0 + V * c, V, cols))
        return out, ft
    for lane in range(64):
        q, r = lane % p["dpr"], lane // p["dpr"]
        if not (r < p["rows_per_it"] and npd * q < ft):
            continue
        nval = min(npd, ft - npd * q) if p["ragged"] else npd
        back = npd - nval
        cols = [npd * q + c + (4 * (q >> 2) if p["pad16"] else 0) for c in range(nval)]
        out.append(((f0 + npd * q - back) * bb, 4, cols))
    return out, ft


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}_nb{s[2]}_L{s[3]}_b{s[4]}")
def test_kernel_addresses_stay_inside_their_buffers(shape):
    N, F, nb, L, bb = shape
    rng = np.random.default_rng(F * 7 + nb)
    for key, p in _plans(shape):
        if p["bytewise"]:
            continue                                                 # one load per bin, indexed by (row, feature) directly
        wbytes = 4 if p["acc_width"] == 16 else 8
        row_bytes = F * bb
        for tile in {0, p["n_tiles"] // 2, p["n_tiles"] - 1}:
            lanes, ft = _lane_columns(p, F, bb, tile)
            assert lanes, key
            if p["wide_v"]:   # a matrix that is not 16-byte aligned takes the dword kernel with the same (padded) plan
                lanes = lanes + _lane_columns(p, F, bb, tile, dword_kernel=True)[0]
            for off, nbytes, cols in lanes:
                assert 0 <= off and off + nbytes <= row_bytes, (key, tile, off)       # no load leaves its row
                for col in cols:
                    assert 0 <= col < p["ftp"], (key, tile, col)                       # LDS word inside the bin row
                    assert (nb - 1) * p["ftp"] * wbytes + col * wbytes + wbytes <= p["lds_bytes"]
        # work items of a batched launch: however the rows are spread over the builds, the items fit the table
        for n_builds in {1, 2, min(L, 17), L}:
            for total in {1, 1000, N // 7 + 1, N}:
                t = describe_hist_plan(N, F, nb, L, bb, key[0], key[1], key[2], key[3], rows=total, n_builds=n_builds)["target_rows"] \
                    if n_builds > 1 else None
                if t is None:
                    continue
                cuts = np.sort(rng.integers(0, total + 1, n_builds - 1))
                rows = np.diff(np.concatenate([[0], cuts, [total]]))
                groups = np.maximum(1, -(-rows // t))
                assert int(groups.sum()) <= p["max_items"], (key, n_builds, total, t)
        # slot of the last item a launch can have, and the reduce kernel's walk over the slots
        slots_end = ((p["max_items"] - 1) * p["n_tiles"] + p["n_tiles"] - 1) * p["slot_bytes"] + p["lds_bytes"]
        assert slots_end <= p["partial_bytes"]
        tile_words = nb * p["ftp"]
        xb = -(-tile_words // 256)
        w = np.arange(xb * 256)
        b, f = w // p["ftp"], w % p["ftp"]
        if p["pad16"]:
            g, o = f // 20, f % 20
            f = np.where(o < 16, 16 * g + o, -1)
        for tile in {0, p["n_tiles"] - 1}:
            ftw = min(p["ft"], F - tile * p["ft"])
            ok = (b < nb) & (f >= 0) & (f < ftw)
            assert ok.any()
            assert int(w[ok].max()) * wbytes + wbytes <= p["slot_bytes"]               # word inside the slot
            hoff = b[ok] * F + tile * p["ft"] + f[ok]
            assert 0 <= int(hoff.min()) and int(hoff.max()) < F * nb                   # word inside the histogram
            assert np.unique(hoff).size == hoff.size                                   # every word reduced once


def test_the_launch_shape_of_an_old_unexplained_fault_is_in_bounds():
    # A stand-alone build of 400,000 x 2000 (63 bins, 3-bit) once faulted on the GPU while a development knob forced
    # 196 row groups (16 tiles).  With today's plan for that shape and the forced group count, every slot the
    # kernels and the reduce kernel address lies inside the slot section, every load inside the matrix.
    N, F, nb, L = 400_000, 2000, 63, 63
    p = describe_hist_plan(N, F, nb, L, 1, 3, 3, 0, False, rows=N)
    groups = 196
    assert groups <= p["max_items"]
    lanes = -(-groups // 8) * 8
    grid = lanes * p["n_tiles"]
    seen = set()
    for wg in range(grid):                                           # workgroup -> (tile, row-group lane)
        xcd, s = wg & 7, wg >> 3
        tile, glane = s % p["n_tiles"], (s // p["n_tiles"]) * 8 + xcd
        if glane >= groups:
            continue
        seen.add((glane, tile))
        slot = (glane * p["n_tiles"] + tile) * p["slot_bytes"]
        assert slot + p["lds_bytes"] <= p["partial_bytes"]
    assert len(seen) == groups * p["n_tiles"]                         # every (group, tile) has exactly one workgroup
    rows_per_group = -(-N // groups)
    for item in (0, groups - 1):
        gbegin = min(N, item * rows_per_group); gend = min(N, gbegin + rows_per_group)
        assert gend - gbegin <= p["chunk_rows"]                      # one chunk: handed over with plain stores
        for tile in (0, p["n_tiles"] - 1):
            for off, nbytes, _ in _lane_columns(p, F, 1, tile)[0]:
                assert (gend - 1) * F + off + nbytes <= N * F


@pytest.mark.parametrize("shape", SHAPES + [(9000, F, nb, 31, 2) for F in (8, 9, 10, 13, 26, 41) for nb in (400, 1024)] +
                         [(9000, F, 255, 31, 1) for F in (15, 17, 65, 68, 70, 97, 129)], ids=lambda s: f"{s[0]}x{s[1]}_nb{s[2]}_L{s[3]}_b{s[4]}")
def test_sixteen_byte_pieces_cover_every_bin_of_a_tile_row_once(shape):
    # lane -> (row, piece) of the kernel that reads 16 bytes per lane: loads inside the row, every bin of the tile row in one
    # lane's sixteen (eight) atomics exactly once, whatever the row's rotation of their order
    N, F, nb, L, bb = shape
    for key, p in _plans(shape):
        last = (F - (p["n_tiles"] - 1) * p["ft"]) * bb
        if not (bb == 1 and F % 4 == 0 and p["ft"] == 128 and p["acc_width"] == 32):   # (such tiles, where the rows fill them, stay with the dword kernel)
            assert (p["pieces"] > 0) == (not p["bytewise"] and not p["wide_v"] and last >= 16), key
        if p["pieces"] == 0:
            continue                                                 # other kernels
        P, npd = p["pieces"], 4 // bb
        assert P == -(-p["ft"] * bb // 16)
        rpi = 64 // P
        assert rpi >= 1, key
        for tile in range(p["n_tiles"]):
            f0 = tile * p["ft"]
            ft = min(p["ft"], F - f0)
            for r, turn in itertools.product(range(rpi), {p["turn"], p["contig_turn"]}):
                seen = []
                for c in range(P):
                    if 16 * c >= ft * bb:
                        continue
                    at = min(16 * c, ft * bb - 16)
                    assert 0 <= at and f0 * bb + at + 16 <= F * bb
                    assert at % bb == 0 and (16 * c - at) % bb == 0
                    rot = ((r + c // (2 * bb) * turn) * bb) & 15
                    for i in range(4):
                        for k in range(npd):
                            j = ((i + (rot >> 2)) & 3) * npd + ((k + (rot & 3) // bb) & (npd - 1))
                            if j >= (16 * c - at) // bb:
                                seen.append(at // bb + j)
                assert sorted(seen) == list(range(ft)), (key, tile, r)


@pytest.mark.parametrize("F,nb,bb", [(32, 255, 1), (64, 255, 1), (97, 63, 1), (100, 127, 1), (190, 127, 1), (500, 15, 1), (1017, 63, 1), (1020, 31, 1), (96, 300, 2), (128, 400, 2)])
def test_pieces_spread_over_the_lds_banks(F, nb, bb):
    # a pitch of whole 32 words: the bank of a column is the same in every bin, and the lanes that an LDS atomic serves at once (half a
    # wavefront) meet every bank at most once
    seen = 0
    for (bg, bh), acc in itertools.product(BITS, (16, 32)):
        p = describe_hist_plan(300_000, F, nb, 15, bb, bg, bh, acc)
        P, npd = p["pieces"], 4 // bb
        if P < 32 * bb // 16 or P & (P - 1) or p["ftp"] % 32 or p["ft"] * bb % 16:
            continue
        assert p["turn"] == 32 // P and p["contig_turn"] == (32 // P if p["acc_width"] == 32 or p["lds_bytes"] * 3 > 160 * 1024 or 300_000 * F * bb <= 2 ** 28 else 0)
        seen += 1
        rpi = 64 // P
        for half in (range(32), range(32, 64)):
            for i in range(4):
                for k in range(npd):
                    banks = []
                    for lane in half:
                        c, r = lane % P, lane // P
                        rot = ((r + c // (2 * bb) * p["turn"]) * bb) & 15
                        kk = (k + (rot & 3) // bb) & (npd - 1)
                        banks.append((16 * c // bb + ((i + (rot >> 2)) & 3) * npd + kk) % 32)
                    assert r < rpi and len(set(banks)) == 32, (bg, bh, acc, i, k)
    assert seen or nb == 400


# which widths the piece kernel serves: (tiles, features per tile, pieces); 0 pieces: the last tile is narrower than one
@pytest.mark.parametrize("F,nb,bb,bits,plan", [
    (15, 255, 1, 3, (1, 15, 0)), (16, 255, 1, 3, (1, 16, 1)), (17, 255, 1, 3, (1, 17, 2)), (28, 255, 1, 3, (1, 28, 2)), (50, 255, 1, 4, (1, 50, 4)),
    (68, 255, 1, 3, (2, 40, 3)), (90, 255, 1, 3, (3, 32, 2)), (28, 255, 1, 5, (1, 28, 2)), (36, 255, 1, 5, (2, 20, 2)), (68, 255, 1, 5, (3, 24, 2)),
    (40, 600, 2, 3, (5, 8, 1)), (38, 600, 2, 3, (19, 2, 0)),
    (42, 600, 2, 3, (21, 2, 0)), (44, 600, 2, 3, (11, 4, 0)), (33, 255, 1, 5, (3, 12, 0)), (72, 255, 1, 3, (2, 64, 0))])
def test_widths_that_are_read_in_sixteen_byte_pieces(F, nb, bb, bits, plan):
    p = describe_hist_plan(2_000_000, F, nb, 127, bb, bits, bits)
    assert (p["n_tiles"], p["ft"], p["pieces"]) == plan


@pytest.mark.parametrize("shape", SHAPES + [(16_384, 28, 255, 31, 1), (16_385, 28, 255, 31, 1), (65_536, 68, 255, 31, 1), (65_537, 68, 255, 31, 1),
                                            (30_000, 100, 255, 63, 1), (4100, 28, 255, 31, 1)], ids=lambda s: f"{s[0]}x{s[1]}_nb{s[2]}_L{s[3]}_b{s[4]}")
def test_the_search_adds_up_few_row_groups_only(shape):
    # where a tree's builds are not reduced by a launch of their own, none of them has more than 32 row groups (33 by rounding), whatever the
    # bits and the width allow a group to hold, and however the rows are spread over the builds of a launch
    N, F, nb, L, bb = shape
    for key, p in _plans(shape):
        if p["search_sums"] == 8:
            continue
        assert p["search_sums"] == 2 ** 31 - 1, key
        for n_builds in {1, 2, min(L, 17), L}:
            for total in {1, 700, N // 3 + 1, N}:
                t = describe_hist_plan(N, F, nb, L, bb, key[0], key[1], key[2], key[3], rows=total, n_builds=n_builds)["target_rows"]
                if n_builds > 1 or not p["flat_lanes"]:
                    assert -(-total // t) <= 33, (key, n_builds, total, t)


@pytest.mark.parametrize("F,bb,dwords", [(16, 1, 0), (17, 1, 1), (20, 1, 1), (21, 1, 0), (32, 1, 0), (33, 1, 1), (36, 1, 1), (37, 1, 0), (49, 1, 0), (8, 2, 0), (9, 2, 1),
                                         (10, 2, 1), (11, 2, 0), (17, 2, 1), (19, 2, 0), (25, 2, 0), (28, 1, 0)])
def test_contiguous_rows_of_one_tile_that_are_read_by_dwords(F, bb, dwords):
    # a last piece of one to four bytes of its own, three pieces at most
    for (bg, bh), acc in itertools.product(BITS, (0, 16, 32)):
        p = describe_hist_plan(50_000, F, 255 if bb == 1 else 400, 15, bb, bg, bh, acc)
        if p["n_tiles"] == 1:
            assert p["contig_dwords"] == dwords and p["pieces"] == -(-F * bb // 16), (bg, bh, acc)
        else:
            assert p["contig_dwords"] == 0


# several tiles of 64 or 128 bytes: (pieces, contiguous rows by dwords); both sides of every condition of the rule
@pytest.mark.parametrize("F,nb,bb,acc,plan", [
    (124, 63, 1, 16, (4, 1)), (116, 63, 1, 16, (4, 0)), (100, 63, 1, 16, (4, 0)), (172, 63, 1, 16, (4, 1)), (300, 160, 1, 16, (4, 1)),
    (300, 161, 1, 16, (4, 0)), (300, 63, 1, 32, (4, 0)), (190, 127, 1, 16, (4, 0)), (500, 100, 1, 16, (8, 1)), (500, 127, 1, 16, (8, 0)), (1017, 63, 1, 16, (8, 0)),
    (1020, 63, 1, 32, (0, 1)), (1017, 63, 1, 32, (8, 1)), (128, 257, 2, 16, (4, 1)), (128, 400, 2, 16, (4, 0)), (127, 257, 2, 16, (4, 0)), (60, 300, 2, 16, (4, 1)),
    (56, 300, 2, 16, (4, 0)), (80, 300, 2, 16, (5, 0))])
def test_rows_of_several_tiles_that_are_read_by_dwords(F, nb, bb, acc, plan):
    p = describe_hist_plan(300_000, F, nb, 15, bb, 3, 3, acc)
    assert p["n_tiles"] > 1 and (p["pieces"], p["contig_dwords"]) == plan


def test_small_trees_with_long_row_groups_need_no_reduction():
    rng = np.random.default_rng(0)
    for N in [1, 2, 511, 512, 513, 16_383, 16_384, 16_385, 65_535, 65_536] + rng.integers(1, 140_000, 200).tolist():
        for F, bits in ((28, 2), (28, 5), (68, 3), (100, 3), (100, 8), (500, 4)):
            p = describe_hist_plan(N, F, 255, 31, 1, bits, bits)
            small = N * p["n_tiles"] <= (2 ** 17 if p["n_tiles"] > 1 else 2 ** 14)
            assert p["search_sums"] == (2 ** 31 - 1 if small else 8), (N, F, bits)


# Gathered builds: the row groups that an XCD holds of a build share one stretch of its list and take its blocks in turn (places as
# the library gives them).  Every row once, no group more than a chunk, an XCD's stretches in the order of the XCDs.
@pytest.mark.parametrize("count,groups,item_start,block,chunk", [
    (100_000, 37, 5, 256, 10_000), (100_000, 8, 0, 256, 100_000), (5000, 3, 7, 320, 4681), (257, 2, 6, 256, 600), (1, 1, 3, 512, 1000),
    (20_000, 64, 1, 144, 4000), (1_000_003, 97, 250, 256, 10_922), (9000, 40, 2, 512, 1000), (777, 7, 4, 64, 500), (50_000, 1023, 9, 16, 200)])
def test_row_groups_of_gathered_builds_cover_the_list(count, groups, item_start, block, chunk):
    rows_per_group = -(-count // groups)
    assert rows_per_group + block <= chunk
    seen = np.zeros(count, np.int64)
    begins, members = {}, {}
    for item in range(item_start, item_start + groups):
        first, n, own = describe_row_group(item_start, groups, item)
        assert 0 <= first and 0 <= own < n and first + n <= groups
        x = item % 8
        begin = min(count, first * rows_per_group)
        end = min(count, begin + n * rows_per_group)
        assert begins.setdefault(x, begin) == begin
        members.setdefault(x, []).append(own)
        mine = 0
        for b in range(begin + own * block, end, n * block):
            seen[b:min(end, b + block)] += 1
            mine += min(end, b + block) - b
        assert mine <= chunk
    assert (seen == 1).all()
    assert all(sorted(m) == list(range(len(m))) for m in members.values())
    assert [begins[x] for x in sorted(begins)] == sorted(begins.values())


# Order of the counting pass as the library goes through it: every segment once and with its own node, whatever the nodes' sizes; every
# XCD stays inside its eighth of each node and goes through it in ascending order.  (Steps per eighth: 1, 4 and 8.)
@pytest.mark.parametrize("n_rows,bound", [(3_000_000, True), (7_000_000, True), (3_000_000, False)])
@pytest.mark.parametrize("n_nodes,grid", [(1, 520), (3, 1024), (64, 2048), (65, 2048), (200, 1032), (658, 8)])
def test_counting_pass_takes_every_segment_once(n_nodes, grid, n_rows, bound):
    rng = np.random.default_rng(n_nodes + n_rows)
    n = rng.integers(1, 3 * 1024 // n_nodes + 2, n_nodes)
    n[rng.integers(0, n_nodes)] += 700
    starts = np.concatenate([[0], np.cumsum(n)[:-1]])
    seen = np.zeros(int(n.sum()), np.int64)
    for wg in range(grid):
        last = {}
        for node, seg in describe_segment_order(n_rows, 28, starts, int(n.sum()), wg, grid, bound):
            local = seg - starts[node]
            assert 0 <= local < n[node]
            assert (n[node] * (wg % 8)) // 8 <= local < (n[node] * (wg % 8 + 1)) // 8
            assert last.get(node, -1) < local
            last[node] = local
            seen[seg] += 1
    assert (seen == 1).all()


def test_counting_pass_of_few_segments_goes_from_node_to_node():
    starts = [0, 1, 40, 41]
    got = [p for wg in range(16) for p in describe_segment_order(3_000_000, 28, starts, 511, wg, 16)]
    assert sorted(s for _, s in got) == list(range(511))
    assert all(node == max(i for i in range(4) if starts[i] <= seg) for node, seg in got)


# Launches that count the left rows themselves: items of one chunk, as many as the table has room for.
COUNTING_SHAPES = [(10_000, 28, 63, 15, 1), (100_003, 50, 255, 31, 1), (65_536, 120, 255, 31, 1), (43_690, 90, 255, 63, 1), (1_000_000, 28, 255, 255, 1),
                   (463_715, 90, 255, 255, 1), (200_000, 136, 255, 63, 1), (100_000, 16, 64, 658, 1), (1_700_000, 48, 255, 127, 1), (20_000, 800, 63, 63, 1),
                   # short chunks and few row-group lanes: more items than the table holds, or nearly as many
                   (262_144, 200, 255, 63, 1), (262_144, 150, 255, 255, 1), (150_000, 200, 255, 63, 1),
                   (50_001, 40, 300, 63, 2), (60_000, 56, 255, 15, 1), (65_536, 50, 255, 63, 1), (3000, 4096, 16, 31, 1), (440_000, 200, 255, 255, 1)]


@pytest.mark.parametrize("shape", SHAPES + COUNTING_SHAPES, ids=lambda s: f"{s[0]}x{s[1]}_nb{s[2]}_L{s[3]}_b{s[4]}")
def test_items_of_launches_that_count(shape):
    N, F, nb, L, bb = shape
    checked = 0
    for (bg, bh), acc, bound in itertools.product(BITS + [(6, 6), (7, 2)], (0, 16, 32), (True, False)):
        key = (bg, bh, acc)
        p = describe_hist_plan(N, F, nb, L, bb, *key)
        c = describe_counting(N, F, nb, L, bb, *key, bound)
        if not c["counts"]:
            continue
        assert p["lds_bytes"] <= 64 * 1024 and not p["bytewise"] and c["seg_rows"] == (2048 if N > 1 << 18 else 512)
        whole = -(-N // c["seg_rows"])
        rng = np.random.default_rng(N)
        for n_nodes in {1, 2, min(L, 17), L}:
            for total in {n_nodes, max(n_nodes, whole // 3), whole + n_nodes - 1}:
                segs = rng.multinomial(total - n_nodes, np.ones(n_nodes) / n_nodes) + 1
                k = describe_counting(N, F, nb, L, bb, *key, bound, None, total, n_nodes)["item_segs"]
                assert k >= 1 and k * c["seg_rows"] <= p["single_rows"], key
                assert total <= c["max_seg"] and n_nodes <= c["batch_max"]
                assert (-(-segs // k)).sum() <= p["max_items"], (key, n_nodes, total)
                if c["search_sums"] != 8:   # the split search adds up every build: none of more than 33 groups
                    assert (-(-segs // k)).max() <= 33, (key, n_nodes, total)
        checked += 1
    assert checked > 0 or shape in SHAPES   # (COUNTING_SHAPES are there because they do)


# Up to how many rows times tiles the histogram launches count, bound and not bound, by leaves, tiles and word width; and that they do
# not where the items' one chunk makes a second turn of the lanes that is nearly empty, or a third one (4 bits: 4096 rows per item)
@pytest.mark.parametrize("F,nb,bh,leaves,tiles,bound,unbound", [
    (28, 255, 3, 64, 1, 3_000_000, 3_000_000), (28, 255, 3, 65, 1, 2_000_000, 2_000_000), (28, 255, 8, 513, 1, 1_400_000, 1_400_000),
    (100, 255, 3, 32, 2, 3_000_000, 3_000_000), (100, 255, 3, 255, 2, 2_000_000, 2_000_000), (90, 255, 3, 20, 3, 3_000_000, 3_000_000),
    (90, 255, 3, 255, 3, 2_000_000, 2_000_000), (140, 127, 8, 160, 3, 2_000_000, 2_000_000), (140, 127, 8, 161, 3, 1_400_000, 1_400_000), (512, 15, 8, 63, 2, 900_000, 900_000), (512, 15, 8, 32, 2, 3_000_000, 3_000_000), (768, 15, 8, 63, 3, 2_000_000, 2_000_000),
    (200, 255, 3, 31, 4, 2_000_000, 2_000_000), (136, 255, 8, 12, 5, 3_000_000, 3_000_000), (552, 31, 3, 31, 9, 1_600_000, 1_100_000),
    (2000, 63, 3, 96, 16, 1_600_000, 1_100_000), (2000, 63, 3, 97, 16, 0, 0)])
def test_trees_up_to_the_lines_count(F, nb, bh, leaves, tiles, bound, unbound):
    p = describe_hist_plan(100_000, F, nb, leaves, 1, 3, bh)
    assert p["n_tiles"] == tiles and (p["acc_width"] == 32) == (bh == 8)
    lanes = 256 // tiles // 8 * 8
    for b, line in ((True, bound), (False, unbound)):
        if bh != 8:
            line = min(line, lanes * 10240 * tiles)   # (one turn of the lanes: 10 602 rows are five segments)
        for N in (max(line // tiles, 1000), line // tiles + 1001):
            assert describe_counting(N, F, nb, leaves, 1, 3, bh, 0, b)["counts"] == (N * tiles <= line), (b, N)


@pytest.mark.parametrize("F,nb,tiles", [(28, 255, 1), (90, 255, 3), (400, 63, 4)])
def test_launches_that_count_take_two_turns_at_most(F, nb, tiles):
    turn = (256 // tiles // 8 * 8) * 4096
    for leaves in (15, 32, 33):
        most = min(2 * turn, 2_000_000 // tiles)
        for rows, counts in ((turn, 1), (turn + 1, leaves > 32), (int(1.28 * turn), leaves > 32), (int(1.32 * turn), 1), (int(1.5 * turn), 1), (most, 1), (most + 1, 0)):
            assert describe_counting(rows, F, nb, leaves, 1, 4, 4, 0, True)["counts"] == counts, (rows, leaves)
