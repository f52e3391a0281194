"""What a decode launch consists of, as the library works it out on the host: where its merging and its tracking blocks lie
behind the stream blocks."""
import ctypes as C

import pytest


def _places(lib, units, n_sub, n_split, group, tracking, f32, d, own_lengths=False):
    fn = getattr(lib, "_ZN6lazyev19decode_fused_placesEiiiibbibPiS0_S0_")   # lazyev::decode_fused_places (kernels.h)
    fn.restype, fn.argtypes = None, [C.c_int] * 4 + [C.c_bool, C.c_bool, C.c_int, C.c_bool] + [C.POINTER(C.c_int32)] * 3
    merge, n_merge, track = C.c_int32(-1), C.c_int32(-1), C.c_int32(-1)
    fn(units, n_sub, n_split, group, tracking, f32, d, own_lengths, C.byref(merge), C.byref(n_merge), C.byref(track))
    return merge.value, n_merge.value, track.value


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group", [1, 2, 4, 5, 7, 8])
def test_merging_and_tracking_blocks(lazyev_lib, d, group, f32):
    """Blocks go to the eight XCDs in turn: tracking block i is on the XCD of stream block i where the tracking blocks begin at
    a multiple of eight.  No two kinds of blocks overlap, and no more than seven blocks are left empty.  Merging blocks are
    there where at most one stream block is on a compute unit, and never where two of long runs are on each."""
    for units in range(1, 65):
        for n_split in range(1, 65):
            stream = units * n_split
            for run in (1, 15, 30):
                merge, n_merge, track = _places(lazyev_lib.lib, units, 4 * n_split * run, n_split, group, True, f32, d)
                if n_split <= 8 or (run == 30 and stream > 512 + 25):
                    assert n_merge == 0
                if n_split > 8 and stream <= 256:  # (compute units of the chip, and what is assumed without one)
                    assert n_merge > 0
                if n_merge == 0:
                    assert track == stream
                    continue
                # a wave merges 32 output elements, a block has two or four such waves
                assert n_merge % units == 0 and group * (d // 32) <= n_merge // units * (4 if n_split <= 16 else 2) < group * (d // 32) + 4
                assert track % 8 == 0
                if merge == stream:
                    assert 0 <= track - (stream + n_merge) < 8
                else:                              # merging blocks last, behind as many tracking blocks as stream blocks
                    assert _places(lazyev_lib.lib, units, 4 * n_split * run, n_split, group, False, f32, d)[0] == stream
                    assert 0 <= track - stream < 8 and merge == track + stream and 2 * stream + n_merge > 563


@pytest.mark.parametrize("d,f32", [(128, False), (64, False), (64, True), (128, True)])
def test_nine_to_fifteen_blocks_where_there_is_room(lazyev_lib, d, f32):
    """As many blocks a unit as the chip has room for (up to fifteen), from 44 sub-tiles (nine and ten of 128 x bf16: 46) to
    16384 entries: never a part of the chip idle for a rule about one number of units.  Below, and of up to eight blocks up to 48 sub-tiles, six."""
    fn = getattr(lazyev_lib.lib, "_ZN6lazyev18decode_fused_splitEiibib")    # lazyev::decode_fused_split (kernels.h)
    fn.restype, fn.argtypes = C.c_int, [C.c_int, C.c_int, C.c_bool, C.c_int, C.c_bool]
    for units in range(17, 29):
        for n_sub in (44, 63, 64, 128, 161, 321, 513, 640, 1023):
            want = 6 if n_sub < 46 and units > 23 and not f32 and d == 128 else min(256 // units, (n_sub + 3) // 4)
            assert fn(units, n_sub, f32, d, False) == want, (units, n_sub)
    for units in (29, 30):
        assert [fn(units, n_sub, f32, d, False) for n_sub in (44, 46, 48, 49, 60, 100)] == [6, 6, 6, 8, 8, 8]


@pytest.mark.parametrize("d", [64, 128])
def test_sixteen_to_twentyeight_blocks_where_there_is_room(lazyev_lib, d):
    """fp32 rows: all that there is room for, whatever the number of units, once a wave has two sub-tiles to do with 16.  bf16 rows: so
    from 500 sub-tiles on, but for 17 and 18."""
    fn = getattr(lazyev_lib.lib, "_ZN6lazyev18decode_fused_splitEiibib")
    fn.restype, fn.argtypes = C.c_int, [C.c_int, C.c_int, C.c_bool, C.c_int, C.c_bool]
    for units in range(9, 17):
        for n_sub in (128, 300, 500, 1000, 1500):
            most = 256 // units
            assert fn(units, n_sub, True, d, False) == most
            if n_sub >= 500:
                assert fn(units, n_sub, False, d, False) == (16 if most in (17, 18) else most)


@pytest.mark.parametrize("group", [1, 4, 7, 8])
def test_sequences_of_their_own_lengths(lazyev_lib, group):
    """Merging blocks stay before the tracking blocks, at every length; two blocks per compute unit from 16384 entries on where
    nine have room."""
    fn = getattr(lazyev_lib.lib, "_ZN6lazyev18decode_fused_splitEiibib")
    fn.restype, fn.argtypes = C.c_int, [C.c_int, C.c_int, C.c_bool, C.c_int, C.c_bool]
    for units in range(4, 29):
        for n_sub in (128, 321, 640, 751, 1023, 1024, 1199, 1500):
            n = fn(units, n_sub, False, 128, True)
            if units > 25:
                assert n == (512 // units if n_sub >= 1024 else 9)
            merge, n_merge, track = _places(lazyev_lib.lib, units, n_sub, n, group, True, False, 128, own_lengths=True)
            assert merge == units * n and 0 <= track - (merge + n_merge) < 8


def test_records_of_a_split(lazyev_lib):
    """A record less than blocks up to eight blocks a unit, from nine on one each; an area of 512 blocks and a record more per unit
    at most."""
    of, needed = (getattr(lazyev_lib.lib, n) for n in ("_ZN6lazyev23decode_fused_records_ofEi", "_ZN6lazyev27decode_fused_records_neededEii"))
    assert [of(n) for n in range(1, 65)] == list(range(8)) + list(range(9, 65))
    for units in range(1, 1025):
        assert needed(units, 30000) == of(min(64, -(-512 // units))) and units * needed(units, 30000) < 512 + 64
        for n_sub in (1, 40, 100, 500, 1100, 1800):
            split = getattr(lazyev_lib.lib, "_ZN6lazyev18decode_fused_splitEiibib")
            assert of(split(units, n_sub, False, 128, False)) <= needed(units, 16 * n_sub)
