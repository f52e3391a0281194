"""bench.py --timeline: what it makes of the stamps of launches whose units are finished by their last block, and by blocks of
their own."""
import numpy as np
import pytest

import bench


def _stamps(n_split, units, merging, tracking, launch, at):
    """Stamps as the kernel leaves them: streams of 5 us, rows behind the launch's blocks are an earlier launch's."""
    a = np.zeros((256, 8), dtype=np.int64)
    a[:, 0], a[:, 5], a[:, 7] = 10, 900, 1 | ((launch - 1) << 8)
    n_stream = n_split * units
    for b in range(n_stream):
        fin = b >= n_stream - units and not merging
        a[b] = [at + b, at + 170, at + 500 + b, at + 550 + b, at + 700 if fin else 33, at + 800 if fin else at + 600 + b, b % 8,
                (2 if fin else 1) | (launch << 8)]
    a[1, 1] = 0                                    # (its first wave has no sub-tile)
    for b in range(n_stream, n_stream + merging):
        a[b] = [at + 20, 44, at + 640, at + 680, 55, at + 720, b % 8, 3 | (launch << 8)]
    for b in range(n_stream + merging, n_stream + merging + tracking):
        a[b] = [at + 30, 44, 44, 44, 55, at + 300, b % 8, 4 | (launch << 8)]
    return a


@pytest.mark.parametrize("n_split,merging", [(2, 0), (10, 16)])
def test_summary_by_kind_of_block(n_split, merging):
    units = 8
    samples = [bench.timeline_sample(_stamps(n_split, units, merging, tracking, launch, 1000 * launch))
               for launch, tracking in ((7, 0), (8, n_split * units))]
    assert [len(s["stream"]) for s in samples] == [n_split * units] * 2
    assert [len(s["merging"]) for s in samples] == [merging] * 2 and [len(s["tracking"]) for s in samples] == [0, n_split * units]
    res = bench.timeline_summary(samples, units)
    assert len(res["stream_end_by_block_of_the_unit"]) == n_split
    assert res["stamps"]["end of wave 0's stream"]["max"] == pytest.approx(5.0 + (n_split * units - 1) / 100)
    assert res["stamps"]["first sub-tile multiplied"]["min"] == 1.7
    assert res["tracking_blocks"]["end"]["max"] == 3.0
    if merging:
        assert res["merging_blocks"]["all there"]["max"] == 6.8 and res["finishing_blocks"]["stream end"] == {}
        assert res["per_launch"]["last merging block's end - latest stream end"] == pytest.approx(7.2 - 5.0 - (n_split * units - 1) / 100)
        assert res["last_block_of_a_launch"]["finishes_its_unit"] == 0
    else:
        assert res["merging_blocks"]["end"] == {} and res["finishing_blocks"]["block end - partials complete"]["max"] == 1.0
        assert res["last_block_of_a_launch"]["finishes_its_unit"] == 1


def test_no_stamps():
    assert bench.timeline_sample(np.zeros((256, 8), dtype=np.int64)) is None
