"""What the bf16 kernel is given: records of 128 or 256 query rows (with the block-granular band's blocks of 256 rows), their
schedule at the kernel's own costs on 512 or 256 workgroups, and how a schedule is corrected from its launches' times."""
import numpy as np
import pytest

import internal as I
from paper_2503_22796_amd import binding as B
from paper_2503_22796_amd import workloads as W
from test_worklist import _check_schedule

FULL, ARROW, CACHE = 0, 1, 2
BN, BAND_ROWS = 64, 256


def _kept(mode, w, n_text, n_img, image_first, block_band):
    """Boolean [N, N]: the pairs the operator keeps."""
    N = n_text + n_img
    i = np.arange(N)
    img = (i < n_img) if image_first else (i >= n_text)
    both = img[:, None] & img[None, :]
    if mode == FULL or w >= n_img - 1:
        return np.ones((N, N), bool)
    keep = ~both | (np.abs(i[:, None] - i[None, :]) <= w)
    if block_band:
        dense = np.zeros_like(keep)
        for i0 in range(0, N, BAND_ROWS):
            for j0 in range(0, N, BN):
                if keep[i0:i0 + BAND_ROWS, j0:j0 + BN].any():
                    dense[i0:i0 + BAND_ROWS, j0:j0 + BN] = True
        keep = dense
    return keep


@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("flags", [0, 1, 2, 3])
@pytest.mark.parametrize("n_text,n_img", [(0, 1), (1, 127), (100, 155), (130, 126), (127, 130), (200, 600), (333, 900), (64, 0)])
def test_records_of_the_kernel_match_brute_force(rows, flags, n_text, n_img):
    N, image_first, block_band = n_text + n_img, bool(flags & B.DIFA_FLAG_IMAGE_FIRST), bool(flags & B.DIFA_FLAG_BLOCK_BAND)
    hp, win = [FULL, ARROW, ARROW, CACHE, ARROW, ARROW], [0, 0, 63, 0, 64, 129]
    items = I.records(2, hp, win, n_text, n_img, rows, 128, flags)
    n_q, n_kv = -(-N // rows), -(-N // BN)
    assert [(int(r["bh"]), int(r["q_tile"])) for r in items] == [(b * 6 + h, t) for b in range(2) for h in range(6) if hp[h] != CACHE
                                                                for t in range(n_q)]
    rot = n_img // BN if image_first and n_text > 0 and n_img > 0 else 0
    kept = {h: _kept(hp[h], win[h], n_text, n_img, image_first, block_band) for h in range(6) if hp[h] != CACHE}
    for r in items:
        k = kept[int(r["bh"]) % 6][r["q_tile"] * rows:(r["q_tile"] + 1) * rows]
        order = list(range(0, r["kv0_end"])) + list(range(r["kv1_begin"], r["kv1_end"]))
        visited = [(u + rot) % n_kv for u in order]
        assert len(visited) == r["n_tiles"] == len(set(visited))
        some = {t for t in range(n_kv) if k[:, t * BN:(t + 1) * BN].any()}
        assert some <= set(visited)
        if block_band or image_first or int(r["window"]) < 0:
            extra = set()
        else:                                   # a record with text rows or a tile shared by text and image: exactly these
            extra = set(visited) - some
        assert set(visited) == some | extra and len(extra) <= 1
        for u in order:
            t = (u + rot) % n_kv
            free = u < r["nm0_end"] if u < r["kv0_end"] else r["nm1_begin"] <= u < r["nm1_end"]
            if free:                            # nothing to mask: every row of the record keeps every key of the tile
                assert (t + 1) * BN <= N and k[:, t * BN:(t + 1) * BN].all()
    # most tiles of a full head, and of a band much wider than a record, are known to be mask-free
    for r in items:
        if hp[int(r["bh"]) % 6] == FULL:
            free = min(r["nm0_end"], r["kv0_end"]) + max(0, r["nm1_end"] - r["nm1_begin"])
            assert free >= r["n_tiles"] - 1


LAYERS = [W.flux_1k, W.flux_2k_mixed, W.flux_2k_full, W.sd3_1k, W.sd3_2k, W.video_like]


@pytest.mark.parametrize("layer", LAYERS, ids=lambda f: f.__name__)
@pytest.mark.parametrize("speeds", [None, [1.04, 0.97, 1.0, 1.01, 0.98, 1.03, 0.96, 1.01]])
@pytest.mark.parametrize("flags", [0, 1])
def test_schedule_of_the_kernel_covers_every_position_once(layer, speeds, flags):
    wl = layer()
    for rows, n_wg in ((128, 512),) if wl.D == 64 else ((128, 512), (256, 256)):
        items = I.records(wl.B, wl.head_plan, wl.window, wl.n_text, wl.n_img, rows, wl.D, flags)
        segs, wg_begin, merges, n_slots, span, _ = I.schedule(items, wl.D, n_wg, 8, speeds)
        _check_schedule(items, segs, wg_begin, merges, n_slots, n_wg, 8)
        assert n_slots * rows * (wl.D + 2) * 4 <= 68157440          # fits the library's file-scope scratch
        # dies get work in proportion to their speeds: the last one is predicted to finish within 8 % of the mean (a die's
        # plan ends within a few percent of the load it was given, and shares more than 3 % apart are corrected once)
        done = span / (np.asarray(speeds) if speeds else np.ones(8))
        assert done.max() <= 1.08 * done.mean(), (wl.name, rows, done)


@pytest.mark.parametrize("n_cut", [0, 1])
def test_schedule_of_a_few_records(n_cut):
    # fewer records than workgroups: one each, and a long one is cut only where that ends earlier
    n_img = 4096 if n_cut else 200
    items = I.records(1, [FULL, CACHE], [0, 0], 16, n_img, 128, 64)
    segs, wg_begin, merges, n_slots, _, _ = I.schedule(items, 64, 512)
    _check_schedule(items, segs, wg_begin, merges, n_slots, 512, 8)
    assert (len(merges) > 0) == bool(n_cut)
    if not n_cut:
        assert np.diff(wg_begin).max() == 1


# ----------------------------------------------------------------------------- a schedule's correction
SPAN = [1000] * 8
EVEN = [50000.0] * 8
UNEVEN = [50000.0] * 7 + [54000.0]


def test_a_schedule_whose_dies_finish_together_stays():
    version, speeds = I.trial(SPAN, [EVEN], 80)
    assert (version == 0).all() and (speeds == 1.0).all()


def test_a_better_schedule_replaces_one_whose_dies_finish_apart():
    version, speeds = I.trial(SPAN, [UNEVEN, EVEN], 80)
    assert list(version[:4]) == [0, 0, 0, 1] and (version[3:] == 1).all()
    assert speeds[3, 7] < 0.95 < 1.0 < speeds[3, 0]              # the die that finished last gets less
    assert abs(speeds[3].mean() - 1.0) < 0.01


def test_a_slower_schedule_gives_way_to_the_one_before_it_for_good():
    worse = [x * 1.05 for x in UNEVEN]
    version, speeds = I.trial(SPAN, [UNEVEN, worse, UNEVEN], 80)
    assert list(version[3:6]) == [1, 1, 1] and (version[6:] == 2).all()
    assert (speeds[6:] == speeds[0]).all()


def test_no_schedule_is_made_more_than_four_times_again():
    better = [[x * f for x in UNEVEN] for f in (1.0, 0.95, 0.9, 0.85, 0.8)]
    version, _ = I.trial(SPAN, better, 200)
    assert list(np.flatnonzero(np.diff(version)) + 1) == [3, 6, 22]     # after 3, 3 and 16 launches; 32 more settle it
    better[3] = UNEVEN                                                  # ... or show that the one before was faster
    version, speeds = I.trial(SPAN, better, 200)
    assert list(np.flatnonzero(np.diff(version)) + 1) == [3, 6, 22, 54]
    assert (speeds[54:] == speeds[21]).all()


def test_dies_that_are_hardly_busy_settle_at_once():
    version, _ = I.trial([100] * 8, [UNEVEN], 80)                # spans too short to say anything about a rate
    assert (version == 0).all()
    version, _ = I.trial(SPAN, [[500.0] * 7 + [900.0]], 80)
    assert (version == 0).all()


def test_a_schedule_that_a_captured_graph_launches_is_not_made_again():
    # a remake due at the very launch that is captured, and one that would be due later
    for at in (3, 2, 10):
        version, _ = I.trial(SPAN, [UNEVEN, EVEN], 80, capturing=[at])
        before, _ = I.trial(SPAN, [UNEVEN, EVEN], 80)
        assert (version[:at] == before[:at]).all() and (version[at:] == version[at - 1]).all()


def test_resident_schedules_give_way_in_order_of_use_captured_ones_last():
    assert I.victim([1, 1, 0, 1], [0, 0, 0, 0], [4, 1, 9, 2]) == 2          # a free place
    assert I.victim([1, 1, 1, 1], [0, 0, 0, 0], [4, 1, 9, 2]) == 1
    assert I.victim([1, 1, 1, 1], [0, 1, 0, 0], [4, 1, 9, 2]) == 3
    assert I.victim([1, 1, 1, 1], [1, 1, 0, 1], [4, 1, 9, 2]) == 2
    assert I.victim([1, 1, 1, 1], [1, 1, 1, 1], [4, 1, 9, 2]) == 1          # nothing else left


# ----------------------------------------------------------------------------- what compiling a plan takes
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("heads,n_text,n_img", [(4, 16, 64), (6, 77, 400), (24, 77, 256), (24, 0, 512)])
def test_a_layer_whose_records_cannot_be_cut_is_compiled_without_a_search(D, heads, n_text, n_img):
    # records of fewer than 16 key tiles: a piece of a record has at least eight, so every record stays whole; such a layer's
    # first call is shorter than a search for cuts
    hp = [FULL] * (heads // 3) + [ARROW] * (heads - heads // 3)
    items = I.records(1, hp, [0] * (heads // 3) + [30] * (heads - heads // 3), n_text, n_img, 128, D)
    assert items["n_tiles"].max() < 16
    segs, wg_begin, merges, n_slots, _, tried = I.schedule(items, D, 512)
    _check_schedule(items, segs, wg_begin, merges, n_slots, 512, 8)
    assert tried == 0 and n_slots == 0


def test_a_layer_of_mostly_uncuttable_records_is_not_searched_to_the_end():
    # narrow bands at 2K: 12 or 14 key tiles a record but for the text rows' 264; no target load holds everything, and that is
    # found out twice for each die and rule, not four or five times
    items = I.records(1, [ARROW] * 24, [128] * 24, 512, 16384, 128, 128)
    *_, tried = I.schedule(items, 128, 512)
    assert tried <= 2 * 2 * 8


# ----------------------------------------------------------------------------- what a plan object sets aside
def test_schedule_memory_of_a_plan_object():
    # a segment is 64 bytes; at most one for every record, two for every workgroup and an entry of 16 bytes for every two of those
    for tokens, heads in ((4608, 24), (16896, 24), (80, 4)):
        device, pinned, n = I.schedule_memory(1, heads, B.DIFA_DTYPE_BF16, tokens)
        most = (heads * -(-tokens // 128) + 1024) * 64 + 512 * (16 + 4)
        assert n == 32 and most <= device / n <= most + 1024 and pinned == device // n * 16
    # the fp32 path keeps records of 44 bytes, one for 256 rows
    device, pinned, n = I.schedule_memory(1, 24, B.DIFA_DTYPE_F32, 4608)
    assert n == 32 and 24 * 18 * 44 <= device / n <= 24 * 18 * 44 + 1024
    # large layers: bounded, but eight schedules in any case
    device, _, n = I.schedule_memory(2, 64, B.DIFA_DTYPE_BF16, 1 << 18)
    assert 8 <= n < 32 and device <= 256 << 20
    assert I.schedule_memory(2, 128, B.DIFA_DTYPE_BF16, 1 << 22)[2] == 8


# ----------------------------------------------------------------------------- the cached-head copy
def test_cached_heads_of_any_length_can_share_the_fp32_launch():
    # chunks of 8192 vectors of 16 bytes; a head of 2^26 tokens of 128 floats has 2^31 vectors, one more than an int holds
    assert I.copy_chunks(1, 64, B.DIFA_DTYPE_F32, 1, 1) == 1
    assert I.copy_chunks(256, 128, B.DIFA_DTYPE_F32, 2, 3) == 6
    assert I.copy_chunks(257, 128, B.DIFA_DTYPE_F32, 2, 3) == 12
    assert I.copy_chunks(1 << 26, 128, B.DIFA_DTYPE_F32, 1, 1) == 1 << 18
    assert I.copy_chunks((1 << 30) - 1, 128, B.DIFA_DTYPE_F32, 1, 2) == 1 << 23


# ----------------------------------------------------------------------------- which record length
@pytest.mark.parametrize("rows,heads,n_text,n_img,full,w,flags", [
    (256, 24, 512, 8704, 24, 0, 0),          # every head full: nothing to save, from about 1.5 K tokens on
    (256, 24, 77, 1459, 24, 0, 0),
    (256, 24, 512, 12544, 24, 0, 0),
    (128, 24, 77, 691, 24, 0, 0),            # ... but short records, or too few of them, are the better for being shorter
    (128, 6, 77, 1459, 6, 0, 0),
    (256, 24, 512, 16384, 0, 2048, 1),       # blocks of 256 rows are visited whole either way
    (128, 24, 512, 16384, 0, 128, 1),
    (256, 24, 512, 16384, 0, 4224, 0),       # bands so wide that a record's rows hardly count
    (128, 24, 512, 16384, 0, 2112, 0),
    (128, 24, 512, 16384, 0, 128, 0),
    (256, 24, 512, 8704, 12, 576, 0),        # full and arrow heads: by what their records would save
    (128, 24, 512, 8704, 4, 576, 0),
    (128, 4, 16, 64, 2, 8, 0),               # the smallest
])
def test_record_length_at_head_dim_128(rows, heads, n_text, n_img, full, w, flags):
    hp, win = [FULL] * full + [ARROW] * (heads - full), [0] * full + [w] * (heads - full)
    assert I.record_rows(1, 128, hp, win, n_text, n_img, flags) == rows
    assert I.record_rows(1, 64, hp, win, n_text, n_img, flags) == 128


def test_record_length_of_the_named_layers():
    for layer, rows in ((W.flux_1k, 128), (W.flux_2k_mixed, 128), (W.flux_2k_full, 256), (W.video_like, 128), (W.tiny, 128)):
        wl = layer()
        assert I.record_rows(wl.B, wl.D, wl.head_plan, wl.window, wl.n_text, wl.n_img) == rows, wl.name
    wl = W.flux_2k_mixed()
    assert I.record_rows(2, wl.D, wl.head_plan, wl.window, wl.n_text, wl.n_img) == 256          # 16.7 M pairs a compute unit
    assert I.record_rows(1, wl.D, [CACHE] * 24, [0] * 24, wl.n_text, wl.n_img) == 128           # nothing computed


@pytest.mark.parametrize("heads,speeds", [(64, [1.03, 0.97, 1.02, 0.98, 1.0, 1.0, 1.01, 0.99]), (60, [1.1, 0.9, 1.05, 0.95, 1.0, 1.0, 1.0, 1.0])])
def test_speeds_of_dies_do_not_give_one_more_records_than_workgroups(heads, speeds):
    # 512 (or 480) equal records on 512 workgroups: in proportion to the speeds some die would get 65 for its 64 workgroups and
    # take as long as two records
    items = I.records(1, [FULL] * heads, [0] * heads, 0, 1024, 128, 128)
    segs, wg_begin, merges, n_slots, span, _ = I.schedule(items, 128, 512, 8, speeds)
    _check_schedule(items, segs, wg_begin, merges, n_slots, 512, 8)
    one = I.schedule(items, 128, 512)[4].max()
    assert (span / np.asarray(speeds)).max() <= 1.12 * one


@pytest.mark.parametrize("heads,full,w,n_text,n_img", [(18, 2, 256, 77, 2048), (16, 2, 256, 333, 2094), (26, 2, 256, 77, 2897), (32, 16, 256, 333, 2094)])
@pytest.mark.parametrize("speeds", [[1.04, 0.96, 1.03, 0.97, 1.0, 1.01, 0.99, 1.0], [1.06, 0.94, 1.05, 0.95, 1.02, 1.0, 0.98, 1.0]])
def test_no_die_is_left_far_behind_where_another_share_of_the_work_helps(heads, full, w, n_text, n_img, speeds):
    # up to a few records for each workgroup: one way of sharing the work out lets the last die end at 1.5 to 2.2 times the mean
    items = I.records(1, [FULL] * full + [ARROW] * (heads - full), [w] * heads, n_text, n_img, 128, 128)
    segs, wg_begin, merges, n_slots, span, _ = I.schedule(items, 128, 512, 8, speeds)
    _check_schedule(items, segs, wg_begin, merges, n_slots, 512, 8)
    done = span / np.asarray(speeds)
    assert done.max() <= 1.12 * done.mean()


@pytest.mark.parametrize("D,full,windows,n_text,n_img,speeds,bound", [
    (64, 1, [66, 207, 831, 831, 415], 333, 3325, [0.98, 1.051, 1.033, 0.97, 1.05, 0.973, 0.985, 1.007], 4.2),
    (128, 2, [469, 225, 938, 938, 469, 225, 225, 112, 225, 225], 256, 3752, [1.019, 1.016, 0.968, 0.982, 1.024, 1.02, 1.003, 0.967], 2.3),
    (64, 12, [30, 252, 126, 252, 126, 63, 20, 252, 252, 30, 30, 30, 20], 512, 1011, [0.972, 1.011, 0.989, 0.993, 1.04, 1.041, 1.044, 1.009], 2.3)])
def test_equal_shares_do_not_rule_out_the_correction_of_others(D, full, windows, n_text, n_img, speeds, bound):
    # 174, 384 and 300 records on 512 workgroups.  In proportion to the speeds and corrected, the last die ends at 4.19, 2.27 and
    # 2.27 times the iterations shared out evenly over all workgroups; equal shares, which end before the uncorrected ones, at
    # 12.5, 3.20 and 2.35.
    items = I.records(1, [FULL] * full + [ARROW] * len(windows), [0] * full + windows, n_text, n_img, 128, D)
    segs, wg_begin, merges, n_slots, span, _ = I.schedule(items, D, 512, 8, speeds)
    _check_schedule(items, segs, wg_begin, merges, n_slots, 512, 8)
    assert (span / np.asarray(speeds)).max() <= bound * 8 * int(items["n_tiles"].sum()) / (64 * sum(speeds))
