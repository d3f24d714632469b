"""Which division of its work a decode call takes (host only). The host knows a
table's width, not the lengths: beyond widths whose batches are all alike, a
table with room to spare must not change the division."""
import pytest

import paper_2411_01142_amd as neo

WIDE = (200, 256, 257, 512, 2048, 8192)


@pytest.mark.parametrize("batch,hkv,want", [
    (64, 8, "whole"), (512, 1, "whole"), (33, 8, "whole"), (32, 8, "whole"), (200, 1, "whole"),
    (13, 8, "units"), (4, 32, "units"), (16, 8, "units"), (128, 1, "units"), (40, 1, "units"),
    (13, 3, "units"), (1, 8, "pairs"), (1, 1, "pairs"), (1, 128, "pairs"),
    (256, 8, "head_slices"), (512, 8, "head_slices"), (1024, 8, "head_slices"),
    (65, 8, "whole"), (96, 8, "whole"), (128, 6, "whole"), (97, 8, "wave_slices"),
    (129, 5, "wave_slices"), (200, 8, "wave_slices"), (513, 1, "wave_slices"),
    (1024, 1, "wave_slices"), (2048, 1, "wave_slices"), (171, 3, "wave_slices")])
def test_room_in_the_table_does_not_change_the_division(batch, hkv, want):
    got = {w: neo.debug_division(batch, 4 * hkv, hkv, w) for w in WIDE}
    assert set(got.values()) == {want}, got


def test_tables_of_short_pairs_and_small_shares():
    d = neo.debug_division
    # At most 32 blocks a pair, up to three pairs per compute unit.
    assert d(64, 32, 8, 32) == "pairs" and d(64, 32, 8, 33) == "whole"
    assert d(96, 32, 8, 32) == "pairs" and d(97, 32, 8, 32) == "wave_slices"
    assert d(768, 8, 1, 32) == "pairs" and d(768, 8, 1, 33) == "wave_slices"
    assert d(4, 32, 32, 32) == "pairs" and d(4, 32, 32, 33) == "pairs"
    # One workgroup a pair of at most 64 blocks where none can be cut.
    assert d(32, 32, 8, 64) == "pairs" and d(32, 32, 8, 65) == "whole"
    # At most 32 blocks a workgroup of a pair.
    assert d(13, 32, 8, 64) == "pairs" and d(13, 32, 8, 65) == "units"
    assert d(2, 32, 8, 512) == "pairs" and d(2, 32, 8, 513) == "units"


def test_calls_that_keep_wave_slices():
    d = neo.debug_division
    for kw in (dict(variant="valu"), dict(max_slices=1), dict(max_slices=4096)):
        for batch in (1, 13, 64, 512):
            assert d(batch, 32, 8, 128, **kw) == "wave_slices"
    # Head slices: whole groups of four heads, two of them per compute unit, and
    # a table that has room for 64 blocks of them per compute unit.
    assert d(255, 32, 8, 512) == "wave_slices" and d(256, 32, 8, 31) == "wave_slices"
    assert d(256, 32, 8, 32) == "head_slices" and d(512, 24, 6, 512) == "wave_slices"


@pytest.mark.parametrize("cus", [1, 2, 8, 32, 64, 128, 256, 304])
def test_every_device_size_gives_a_division(cus):
    for batch in (1, 2, 7, 64, 513, 5000):
        for hkv in (1, 3, 8, 64):
            for width in (1, 32, 33, 600, 100000):
                if batch * hkv * (width + 3) < 2 ** 31:
                    assert neo.debug_division(batch, hkv, hkv, width,
                                              compute_units=cus) in neo.DIVISIONS


def test_bad_shapes_are_refused():
    for bad in (dict(batch=0), dict(num_kv_heads=3), dict(max_blocks_per_seq=0),
                dict(compute_units=0), dict(max_slices=-1)):
        args = dict(batch=4, num_q_heads=8, num_kv_heads=2, max_blocks_per_seq=10)
        with pytest.raises(neo.NeoError):
            neo.debug_division(**{**args, **bad})
