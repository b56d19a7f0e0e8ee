"""Host rules against plain models, without a GPU."""
import itertools
import random

import numpy as np
import pytest

from tests.rules import lib


@pytest.mark.parametrize("elem", [1, 2, 4])
def test_tap_reach_is_the_last_byte_that_row_indexed_loads_touch(elem):
    """Eight bytes from the pair's aligned dword (f32: from the pair) in rows
    y0 and y0 + 1, over every valid corner."""
    for w, h, pad in itertools.product(range(2, 14), (2, 3, 5), (0, 1, 2)):
        pitch = (w * elem + 3) // 4 * 4 + 4 * pad
        last = 0
        for x0, y in itertools.product(range(w - 1), range(h)):
            col = x0 * elem
            last = max(last, y * pitch + (col if elem == 4 else col // 4 * 4) + 8)
        assert lib().tap_reach(w, h, pitch, elem) == last
        end = lib().image_end(w, h, pitch, elem)
        assert end == (h - 1) * pitch + (w * elem + 3) // 4 * 4
        assert last <= end + 4 and (elem != 4 or last <= end)


@pytest.mark.parametrize("elem,w", [(1, 640), (1, 638), (1, 637), (1, 639), (2, 640), (2, 639), (4, 640)])
def test_rows_are_read_by_index_only_over_mapped_memory(elem, w):
    h = 16
    pitch = (w * elem + 3) // 4 * 4
    end = lib().image_end(w, h, pitch, elem)
    past = lib().tap_reach(w, h, pitch, elem) > end
    assert past == ((elem, w) not in [(1, 637), (2, 639), (4, 640)])

    def safe(data, next_, mapped):
        return bool(lib().rows_by_index_safe(data, w, h, pitch, elem, next_, mapped))
    page = 1 << 32
    at = page - end                       # the image ends with a page
    assert safe(at, 0, page) == (not past)          # and with the mapped memory
    assert safe(at, 0, page + 3) == (not past)
    assert safe(at, 0, page + 4)                    # the dword past it is mapped
    assert safe(at, page, page)                     # the next image starts there
    assert safe(at, page + 4096, page) == (not past)
    assert safe(at - 4, 0, page - 4)                # the dword lies in the last byte's page
    assert safe(at + 4, 0, page + 4)


@pytest.mark.parametrize("f32", [0, 1])
def test_disc_wavefronts_have_slots_to_deal(f32):
    """Several wavefronts share a disc only where it has several pixel slots,
    and take a second round (w > 1) only where each has one of its own."""
    for slots in range(1, 17):
        for w in (0.01, 0.25, 0.26, 0.45, 0.46, 1.0, 1.01, 1.7, 1.71, 2.2, 2.3, 4.0, 4.1, 50.0):
            f = lib().disc_form(w, slots, f32, 0)
            waves, deep, shared = f // 100, f // 10 % 10, f % 10
            assert (waves, deep, shared) in [(16, 4, 0), (8, 4, 0), (4, 4, 0), (1, 4, 0), (1, 2, 1)]
            assert waves == 1 or slots > 1
            assert waves == 1 or waves * w <= 4.0 or slots >= 4
            damped = lib().disc_form(w, slots, f32, 1)
            assert damped // 100 == 1 and damped % 10 == 0


def test_one_workgroup_bins_a_keyframe_only_where_that_is_little_work():
    def lds(*a):
        return bool(lib().bin_in_lds(*a))
    assert lds(1, 1200, 1564) and lds(1, 15360, 3072) and not lds(1, 15361, 10)
    assert not lds(1, 8160, 3073) and not lds(8, 15252, 15252) and not lds(11, 3600, 4641)
    assert lds(12, 3600, 4641) and lds(64, 1200, 6400) and not lds(64, 1200, 6401) and not lds(12, 15361, 1)


def _cut(nq, items, nbr, fixed):
    base = np.concatenate([[0], np.cumsum(items)])
    kfs = np.ascontiguousarray(np.stack([items, nbr, base[:-1]], 1).astype(np.int32))
    out = np.full(2 * nq, -1, np.int32)
    lib().cut_shares(nq, kfs.ctypes.data, len(items), fixed, out.ctypes.data)
    return out, int(base[-1])


@pytest.mark.parametrize("nq", [1, 8])
@pytest.mark.parametrize("fixed", [0.5, 1.0])
def test_item_runs_cover_every_item_once_in_equal_work(nq, fixed):
    """Runs are ordered, meet and cover the items; none is heavier than its
    part of the work by more than one item; the grid of workgroups takes every
    item exactly once."""
    rng = random.Random(nq)
    lists = [[1], [0], [7], [8], [0, 0, 0], [5, 0, 0, 3], [1] * 9, [3000, 1, 1, 1], [1, 1, 3000], [5000] * 3]
    lists += [[rng.randint(0, 10 ** rng.randint(1, 3)) for _ in range(rng.randint(1, 40))] for _ in range(40)]
    for items in lists:
        nbr = [rng.randint(1, 16) for _ in items]
        out, total = _cut(nq, items, nbr, fixed)
        begin, end = out[::2], out[1::2]
        assert begin[0] == 0 and end[-1] == total and (begin[1:] == end[:-1]).all() and (begin <= end).all()
        work = np.repeat(np.array(nbr, float) + fixed, items)
        at = np.concatenate([[0.0], np.cumsum(work)])
        heavy = np.max(work, initial=0.0)
        assert (at[end] - at[begin] <= at[-1] / nq + heavy + 1e-6 * at[-1]).all()
        for wpb in (1, 4):
            blocks = lib().item_blocks(nq, out.ctypes.data, total, wpb)
            seen = np.zeros(total + wpb, int)
            for b in range(blocks):
                if nq == 8:
                    first, last = begin[b % 8] + b // 8 * wpb, end[b % 8]
                else:
                    first, last = b * wpb, total
                seen[first:max(first, min(first + wpb, last))] += 1
            assert (seen[:total] == 1).all() and (seen[total:] == 0).all()


def test_init_reach_counts_the_tiles_that_a_radius_meets():
    for s in (4, 8, 16):
        assert lib().init_reach(0.0, s) == 1 == lib().init_reach(float(s), s) and lib().init_reach(0.1, s) == 0
        for br in (0.7 * s, 1.4 * s, 2.6 * s, 5.1 * s):
            centre = (s - 1) / 2
            met = max(t for t in range(9) if max(0.0, t * s - centre) < br)          # the tile t's nearest pixel
            assert lib().init_reach(br, s) == met
        assert lib().init_reach(3e38, s) > 16384


def test_raster_takes_a_pixel_per_lane_for_few_tiles_with_long_lists():
    """The expected list is the surfels' boxes over the tiles, counted here for
    centres spread evenly over a plane of whole tiles."""
    for r in (0.5, 2.5, 6.0, 12.0):
        at = (np.arange(1600) + 0.5) / 100.0                    # a tile's width of centres
        met = np.floor((at + r) / 16.0) - np.floor((at - r) / 16.0) + 1
        assert abs(met.mean() ** 2 - lib().mean_tiles(r, 16)) < 0.01 * lib().mean_tiles(r, 16)
    assert lib().raster_pixels(1280, 8.0, 256) == 1 and lib().raster_pixels(1, 9.0, 256) == 1
    assert lib().raster_pixels(1281, 500.0, 256) == 4 and lib().raster_pixels(1, 7.9, 256) == 4


@pytest.mark.parametrize("patch", [4, 16])
def test_damped_batches_that_only_seven_wavefronts_per_simd_hold_take_that_form(patch):
    """Between five and seven items per SIMD one round of one sample at a time
    against two of one frame in flight; large images' taps outweigh it for 4x4
    surfels."""
    def one(w, width, height, elem, frames):
        px = width * height
        b = px * elem * (frames + 1)
        return bool(lib().damped_one_frame(w, patch, px, b, frames, elem == 4 or elem == 2 and b > 8e6))
    for w in (5.01, 6.0, 6.2, 6.9, 7.0):
        assert not one(w, 320, 240, 2, 6) and not one(w, 320, 240, 4, 12)
        assert one(w, 640, 480, 4, 6) == (patch == 4) and one(w, 640, 480, 1, 6) == (patch == 4 and w > 6.2)
    for w in (3.01, 4.0, 7.01, 9.0):
        assert one(w, 320, 240, 2, 12) and one(w, 640, 480, 4, 6)
    assert one(5.0, 320, 240, 2, 6) and one(5.0, 320, 240, 2, 12) == (patch == 16)
    for w in (9.01, 24.0, 24.1, 100.0):
        assert not one(w, 320, 240, 2, 6) and one(w, 640, 480, 4, 6) and one(w, 640, 480, 2, 6) == (w <= 24.0)
