"""The form in which a call runs the chunkwise linear branch, on both sides of the lines between the forms: in segments (how many), or in
one pass with one or two slices of 16 value columns per block.  (Decided on the host; nothing is launched.)"""
import ctypes

import pytest

from paper_2602_03681_amd import binding as nb

from test_segment_rule import segments


def form(H, chunks, d, dtype=nb.NATS_BF16, **kw):
    return nb.linear_scan_form(nb.make_fwd_params(1, H, 64 * chunks, d, 64, dtype, **kw))


@pytest.mark.parametrize("d,H,chunks,want", [
    # one slice per block as long as the heads' slices fit the CUs (32 heads of 128 columns, 64 of 64), up to the length from which
    # two passes over segments are shorter ...
    (128, 1, 1, (1, 1)), (128, 2, 39, (1, 1)), (128, 2, 40, (10, 0)), (128, 18, 39, (1, 1)), (128, 18, 40, (10, 0)),
    (128, 32, 47, (1, 1)), (128, 32, 48, (8, 0)),
    (64, 1, 1, (1, 1)), (64, 2, 31, (1, 1)), (64, 2, 32, (8, 0)), (64, 32, 37, (1, 1)), (64, 32, 38, (8, 0)),
    # (33 to 64 heads of 64 columns: one pass up to 68 or 88 chunks)
    (64, 40, 68, (1, 1)), (64, 40, 69, (6, 0)), (64, 40, 256, (6, 0)), (64, 48, 88, (1, 1)), (64, 48, 89, (5, 0)), (64, 64, 88, (1, 1)),
    (64, 64, 89, (4, 0)), (64, 64, 384, (4, 0)), (64, 65, 384, (1, 2)),
    # ... then two ...
    (128, 33, 27, (1, 2)), (128, 33, 28, (7, 0)), (128, 48, 64, (1, 2)), (128, 48, 65, (5, 0)), (128, 64, 64, (1, 2)),
    (64, 64, 32, (1, 1)), (64, 65, 32, (1, 2)), (64, 128, 64, (1, 2)),
    # ... and beyond 64 (128) heads segments: one, or three
    (128, 65, 17, (1, 0)), (128, 65, 18, (3, 0)), (128, 96, 64, (1, 0)), (64, 136, 32, (1, 0)),
    # whatever the length and however many: slices in several rounds of blocks are not taken
    (128, 128, 136, (1, 0)), (128, 128, 512, (1, 0)), (128, 320, 32, (1, 0)), (128, 576, 32, (1, 0)),
    (64, 136, 512, (1, 0)), (64, 264, 32, (1, 0)), (64, 320, 8, (1, 0)), (64, 512, 32, (1, 0)), (64, 704, 256, (1, 0)),
])
def test_lines(d, H, chunks, want):
    assert form(H, chunks, d) == want


@pytest.mark.parametrize("H,chunks,d", [(18, 67, 128), (1, 128, 128), (24, 51, 64), (40, 35, 128)])
def test_no_more_segments_than_the_workspace_has_room_for(H, chunks, d):
    n, slices = form(H, chunks, d)
    assert slices == 0 and 1 < n <= segments(H, 64 * chunks, d)


def test_groups_count_output_heads():
    for chunks in (47, 48):
        assert form(16, chunks, 128, group=2) == form(32, chunks, 128)
    assert form(11, 8, 128, group=3) == form(48, 8, 128) == (1, 2)


def test_a_given_number_means_segments():
    assert form(2, 16, 128, gdn_segments=4) == (4, 0) and form(2, 1, 64, gdn_segments=8) == (1, 0)
    assert form(3, 22, 64, gdn_segments=5) == (5, 0) and form(3, 19, 64, gdn_segments=4) == (4, 0)
    assert form(3, 28, 64, gdn_segments=6) == (6, 0) and form(3, 34, 64, gdn_segments=8) == (7, 0)   # (no empty segment)


def test_other_paths_have_no_form():
    assert form(2, 16, 128, dtype=nb.NATS_F32) == form(2, 16, 128, math=nb.NATS_MATH_FP32) == (0, 0)
    assert nb.linear_scan_form(nb.make_fwd_params(1, 2, 1024, 128, 128, nb.NATS_BF16, routing=nb.NATS_ROUTE_CHUNK)) == (0, 0)


def test_refusals():
    lib = nb.load_library()
    n = ctypes.c_int32()
    assert lib.nats_linear_scan_form(ctypes.byref(nb.make_fwd_params(1, 2, 1024, 128, 64, nb.NATS_BF16)), None, ctypes.byref(n)) == -1
    with pytest.raises(nb.NatsError):
        form(2, 16, 96)
