"""What a frame reserves (host arithmetic, no GPU)."""
import ctypes

import pytest

from paper_2411_02703_amd import binding as B
from paper_2411_02703_amd import scenes


def _bytes(w, h, seg_len):
    o = B.default_opts(tile_w=8, tile_h=8, seg_len=seg_len)
    cams = B.make_cameras([scenes.identity_camera(50.0, 50.0, w / 2, h / 2, w, h)])
    assert B.load().gs_plan_cameras(cams, 1, ctypes.byref(o)) == 0
    return B.load().gs_frame_bytes(1000, cams, 1, ctypes.byref(o), 10_000)


@pytest.mark.parametrize("seg_len", [-1, 64, 512])
def test_only_frames_that_split_lists_reserve_state_for_whole_tiles(seg_len):
    """From 2048 tiles on a split frame holds six floats a pixel for the whole tiles of its backward; a frame whose lists are
    never split runs a backward that has no use for them."""
    few, many = _bytes(184, 712, seg_len), _bytes(256, 512, seg_len)  # 2047 and 2048 tiles of 8x8
    state = 2048 * 6 * 64 * 4
    if seg_len < 0:
        assert many - few < state // 8
    else:
        assert state <= many - few < state + state // 8
