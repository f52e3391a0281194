"""What a decode launch consists of, as the library works it out on the host: where its merging and its tracking blocks lie
behind the stream blocks."""
import ctypes as C

import pytest


def _places(lib, units, n_split, group, d):
    fn = getattr(lib, "_ZN6lazyev19decode_fused_placesEiiiiPiS0_S0_")   # lazyev::decode_fused_places (kernels.h)
    fn.restype = None
    merge, n_merge, track = C.c_int32(-1), C.c_int32(-1), C.c_int32(-1)
    fn(units, n_split, group, d, C.byref(merge), C.byref(n_merge), C.byref(track))
    return merge.value, n_merge.value, track.value


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group", range(1, 9))
def test_tracking_blocks_run_on_the_xcds_of_the_stream_blocks(lazyev_lib, d, group):
    """Blocks go to the eight XCDs in turn: tracking block i is on the XCD of stream block i where the tracking blocks begin at
    a multiple of eight.  No two kinds of blocks overlap, and no more than seven blocks are left empty."""
    for units in range(1, 65):
        for n_split in range(1, 65):
            stream = units * n_split
            merge, n_merge, track = _places(lazyev_lib.lib, units, n_split, group, d)
            if n_split <= 8:
                assert (n_merge, track) == (0, stream)
                continue
            # a wave merges 32 output elements, a block has two or four such waves
            assert n_merge % units == 0 and group * (d // 32) <= n_merge // units * (4 if n_split <= 16 else 2) < group * (d // 32) + 4
            assert merge == stream and 0 <= track - (stream + n_merge) < 8 and track % 8 == 0
