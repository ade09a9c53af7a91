"""The benchmark's stage roofline of a render that is binned in two levels (host
arithmetic only): the slots' one-word rectangles, the (slot, cell) pairs and the
lists written once, and nothing of a sort of every instance."""
import types

import numpy as np
import pytest

import bench


def _scene(n):
    means = np.zeros((n, 3), np.float32)
    means[:, 2] = np.linspace(2.0, 3.0, n)
    return types.SimpleNamespace(n=n, means=means, sh_degree=0)


def _cam(w, h):
    return types.SimpleNamespace(R=np.eye(3, dtype=np.float32), t=np.zeros(3, np.float32),
                                 znear=0.01, width=w, height=h)


def _brute_pairs(rects, w, h):
    pairs = set()
    for i, (x0, x1, y0, y1) in enumerate(rects):
        if x0 >= 0:
            pairs |= {(i, x // w, y // h) for x in range(x0, x1 + 1) for y in range(y0, y1 + 1)}
    return len(pairs)


@pytest.mark.parametrize("tiles_x, tiles_y, cell", [
    (32, 16, None),          # 512 tiles: emitted
    (33, 16, (4, 4)),
    (120, 68, (4, 4)),       # 30 x 17 cells
    (121, 68, (8, 4)),       # one column of cells more than 4x4 tiles allow
    (240, 135, (8, 8)),
    (241, 135, None),        # more than 512 cells of 8x8 tiles: emitted
])
def test_cell_pairs(tiles_x, tiles_y, cell):
    rng = np.random.default_rng(tiles_x)
    x0, y0 = rng.integers(0, tiles_x, 200), rng.integers(0, tiles_y, 200)
    rects = np.stack([x0, np.minimum(x0 + rng.integers(0, 12, 200), tiles_x - 1),
                      y0, np.minimum(y0 + rng.integers(0, 12, 200), tiles_y - 1)], 1)
    rects[::7] = -1
    want = None if cell is None else _brute_pairs(rects, *cell)
    assert bench.cell_pairs(rects, tiles_x, tiles_y) == want


@pytest.mark.parametrize("width, rect", [(2032, 4), (2033, 8)])
def test_stage_bytes_in_two_levels(width, rect):
    n, height = 1000, 800
    T = -(-width // 16) * 50
    M, pairs = 5000, 1300
    st = dict.fromkeys(("project", "depth_sort", "emit", "tile_sort", "ranges", "composite"), 0.01)
    conf = {"sort_order": "depth_first", "schedule": "queue", "tile": (16, 16)}
    r = bench.stage_roofline(0, _scene(n), _cam(width, height), conf, (M, T), 100, st, 1e-4, pairs)
    b = {k: v["bytes"] for k, v in r["stages"].items()}
    assert b["project"] == (56 + 12) * n + (52 + rect) * n
    assert b["depth_sort"] == 16 * n * 3 + 2 * rect * n
    assert b["emit"] == 2 * rect * n + 4 * n + 6 * pairs
    assert b["tile_sort"] == 8 * pairs + 4 * M + 8 * T
    assert b["ranges"] == 12 * T
    assert r["tile_sort_passes"] == 0
    # no order under the tile schedule; tile first sorts each tile's list by depth
    r = bench.stage_roofline(0, _scene(n), _cam(width, height), dict(conf, schedule="tiles"),
                             (M, T), 100, st, 1e-4, pairs)
    assert r["stages"]["ranges"]["bytes"] == 0
    r = bench.stage_roofline(0, _scene(n), _cam(width, height),
                             dict(conf, schedule="tiles", sort_order="tile_first"),
                             (M, T), 100, st, 1e-4, pairs)
    b = {k: v["bytes"] for k, v in r["stages"].items()}
    assert b["depth_sort"] == 0 and b["emit"] == 2 * rect * n + 6 * pairs
    assert b["ranges"] == (16 * 3 + 4) * M
