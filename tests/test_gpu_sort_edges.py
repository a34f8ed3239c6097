"""Depth and tile sorts on both sides of the sizes where a launch changes shape: 2^19 items (above, histograms are
scanned in a launch of their own) and 2^23 (above, blocks of 4096 items), more than 2^22 tiles (ids of three digits),
and more blocks of either sort than its launches have workgroups."""
import pytest
import torch

import test_gpu_sort as base
from gpu_helpers import instance_lists, say
from test_gpu_sort import r  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,depths,w,h,views", [((1 << 19) - 1, "wide", 640, 480, 1), (1 << 19, "wide", 640, 480, 1),
                                                ((1 << 19) + 1, "linear", 640, 480, 1), (1 << 21, "wide", 320, 240, 4),
                                                (((1 << 23) + 1) // 3, "wide", 320, 240, 3),
                                                (3000, "linear", 16384, 16384, 1),
                                                # more blocks than a launch has workgroups
                                                (2_900_001, "wide", 320, 240, 6)])
def test_depth_sort_and_tile_digits(r, n, depths, w, h, views):  # noqa: F811
    base.test_sorted_order_and_lists(r, n, depths, w, h, views)


def test_lists_by_capacity(r):  # noqa: F811
    """The launches of the emission and the tile sort follow the capacity: the same lists on either side of each edge."""
    g, _ = base._scene(20000, "linear", 7)
    cam = dict(w2c=[[1.0, 0, 0, 0], [0, 1.0, 0, 0], [0, 0, 1.0, 0]], fx=512.0, fy=512.0, cx=320.0, cy=240.0, width=640,
               height=480)
    opts = dict(tile_w=8, tile_h=8)
    want = None
    for cap in (1 << 19, (1 << 19) + 1, 1 << 23, (1 << 23) + 1, 1 << 26):
        say(f"case lists at capacity {cap}")
        buf, ws = r.new_workspace(20000, [cam], cap, 0, opts)
        r.render_into(g, [cam], r.allocate_outputs([cam]), ws, opts)
        ok, need = r.status(ws)
        assert ok and 4096 < need <= 1 << 19
        got = instance_lists(buf, r.layout(20000, [cam], cap, 0, opts), with_bands=True)
        want = want or got
        assert all((a == b).all() for a, b in zip(want, got))
