"""Depth and tile sorts of the binning at the sizes where a pass changes shape:
one workgroup and its edges, the largest sort without a scan launch and the
next one, depth ranges from one key to every exponent, and tile counts of
one, two and three digits."""
import numpy as np
import pytest
import torch

from gpu_helpers import instance_lists, listed_count, read, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def r():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_18682_amd import renderer as R

    rr = R.Renderer(0)
    yield rr
    rr.close()


def _scene(n, depths, seed):
    """Gaussians of about a pixel spread over the view of an identity camera."""
    rng = np.random.default_rng(seed)
    if depths == "same":
        z = np.full(n, 3.0)
    elif depths == "wide":
        z = np.exp(rng.uniform(np.log(0.21), np.log(1e30), n))
    else:
        z = rng.uniform(1.0, 20.0, n)
    z = z.astype(np.float32)
    z64 = z.astype(np.float64)
    means = np.stack([rng.uniform(-0.55, 0.55, n) * z64, rng.uniform(-0.45, 0.45, n) * z64, z64])
    scales = np.log(0.003 * z64)[None] + rng.normal(0, 0.2, (3, n))
    g = dict(means=means, log_scales=scales, quats=rng.standard_normal((4, n)),
             opacity_logits=rng.normal(0, 1, n), sh=rng.normal(0, 0.3, (1, 3, n)))
    g = {k: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).cuda() for k, v in g.items()}
    return dict(g, sh_degree=0), z


CASES = [(1, "linear", 64, 48, 1), (2047, "same", 320, 240, 1), (2048, "wide", 8, 8, 1), (2049, "linear", 640, 480, 1),
         (4097, "wide", 1000, 900, 2), (40000, "linear", 5000, 4300, 1), ((1 << 20) - 1, "linear", 640, 480, 1),
         ((1 << 20) + 1, "wide", 640, 480, 1), (700_000, "wide", 1024, 1024, 3),
         # one workgroup for the depth order (up to 4096 Gaussian-views), and for the tile order (up to 1024 tiles)
         (1024, "linear", 256, 256, 1), (1025, "wide", 264, 256, 1), (4096, "same", 256, 256, 1),
         (2048, "wide", 128, 128, 2), (4097, "linear", 100, 75, 1), (256, "wide", 100, 75, 1), (257, "wide", 64, 48, 2)]


@pytest.mark.parametrize("n,depths,w,h,views", CASES)
def test_sorted_order_and_lists(r, n, depths, w, h, views):
    say(f"case sort n {n} depths {depths} {w}x{h} x{views}")
    g, z = _scene(n, depths, 7)
    cam = dict(w2c=np.eye(3, 4), fx=0.8 * w, fy=0.8 * w, cx=w / 2, cy=h / 2, width=w, height=h)
    cams = [cam] * views
    opts = dict(tile_w=8, tile_h=8)
    outs, (buf, ws) = r.render(g, cams, opts, keep_workspace=True)
    lay = r.layout(n, cams, ws.capacity, 0, opts)
    counts = read(buf, lay.tile_counts, n * views, np.uint32)
    kept = np.nonzero(counts)[0]
    c = read(buf, lay.counters, 8, np.int64)
    assert c[4] == len(kept) and c[0] == counts.astype(np.int64).sum()
    key = z.view(np.uint32)[kept % n]
    want = kept[np.argsort(key, kind="stable")]
    order = read(buf, lay.order, len(kept), np.uint32)
    assert np.array_equal(order, want)
    assert np.array_equal(read(buf, lay.depth_keys, len(kept), np.uint32), np.sort(key))
    tiles, ids = instance_lists(buf, lay)
    assert listed_count(buf, lay) == len(tiles) and (len(tiles) > 0 or n == 1)
    place = np.zeros(n * views, np.int64)
    place[order] = np.arange(len(order))
    # by tile, then by depth order; no instance twice
    both = tiles * (n * views) + place[ids]
    assert np.all(np.diff(both) > 0)
    rng = read(buf, lay.tile_ranges, 2 * lay.total_tiles, np.uint32).reshape(-1, 2).astype(np.int64)
    assert np.array_equal(rng[:, 1] - rng[:, 0], np.bincount(tiles, minlength=lay.total_tiles))


@pytest.mark.parametrize("tile", [(8, 8), (8, 16), (16, 16), (32, 8), (32, 32)])
@pytest.mark.parametrize("kind", ["tiny", "wide", "mixed"])
def test_emission_lists(r, kind, tile):
    """Rows of one tile, rows across the whole view and both in one frame, at
    capacities just above the need (the fewest blocks) and far above it: the
    same lists, and those of the oracle."""
    import oracle
    import scenegen

    say(f"case emission {kind} {tile}")
    n = {"tiny": 3000, "wide": 150, "mixed": 1200}[kind]
    sc = scenegen.tiny_scene(23, n, half_extent=1.0, log_scale_mean={"tiny": -6.0, "wide": -0.7, "mixed": -4.0}[kind],
                             log_scale_std={"tiny": 0.2, "wide": 0.4, "mixed": 1.6}[kind])
    cam = scenegen.pinhole(scenegen.look_at((0.2, 0.1, -3.0)), 611, 389, 60.0)
    opts = scenegen.default_options(tile_w=tile[0], tile_h=tile[1])
    g = {k: torch.from_numpy(np.ascontiguousarray(sc[k])).cuda() for k in
         ("means", "log_scales", "quats", "opacity_logits", "sh")}
    g["sh_degree"] = sc["sh_degree"]
    _, (buf, ws) = r.render(g, [cam], opts, keep_workspace=True)
    need = r.status(ws)[1]
    got = []
    for cap in (need, need + 1, 2 * need + 77, (1 << 20) + need):
        buf, ws = r.new_workspace(n, [cam], cap, 0, opts)
        outs = r.allocate_outputs([cam])
        r.render_into(g, [cam], outs, ws, opts)
        assert r.status(ws) == (True, need)
        lay = r.layout(n, [cam], cap, 0, opts)
        got.append(instance_lists(buf, lay, with_bands=True))
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)
    sp = oracle.preprocess(sc, cam, opts)
    tiles, _, ids = oracle.tile_lists(sp, cam, opts, 0)
    bad = np.nonzero(sp["hazard"] != 0)[0]
    ok, keep = ~np.isin(got[0][1], bad), ~np.isin(ids, bad)
    assert np.array_equal(got[0][0][ok], tiles[keep]) and np.array_equal(got[0][1][ok], ids[keep])


@pytest.mark.parametrize("tile", [(8, 16), (16, 8)])
@pytest.mark.parametrize("n,size", [(40, 900), (600, 900), (2500, 1500)])
def test_sparse_segments(r, n, size, tile):
    """Thin diagonal needles: most box tiles are not listed, so the tile sort takes
    many emission blocks (from one window's few to hundreds of windows) together."""
    import oracle
    import scenegen

    say(f"case sparse n {n} size {size} {tile}")
    sc = scenegen.tiny_scene(31, n, half_extent=0.8, log_scale_mean=-7.0, log_scale_std=0.2)
    sc["log_scales"] = np.ascontiguousarray(sc["log_scales"])
    sc["log_scales"][0] = -0.9  # one long axis
    cam = scenegen.pinhole(scenegen.look_at((0.2, 0.1, -3.0)), size, size - 37, 60.0)
    opts = scenegen.default_options(tile_w=tile[0], tile_h=tile[1])
    g = {k: torch.from_numpy(np.ascontiguousarray(sc[k])).cuda() for k in
         ("means", "log_scales", "quats", "opacity_logits", "sh")}
    g["sh_degree"] = sc["sh_degree"]
    _, (buf, ws) = r.render(g, [cam], opts, keep_workspace=True)
    need = r.status(ws)[1]
    for cap in (need, 2 * need + 77, (1 << 20) + need):
        buf, ws = r.new_workspace(n, [cam], cap, 0, opts)
        r.render_into(g, [cam], r.allocate_outputs([cam]), ws, opts)
        assert r.status(ws) == (True, need)
        lay = r.layout(n, [cam], cap, 0, opts)
        got = instance_lists(buf, lay, with_bands=True)
        assert len(got[0]) < 0.5 * need
        sp = oracle.preprocess(sc, cam, opts)
        tiles, _, ids = oracle.tile_lists(sp, cam, opts, 0)
        bad = np.nonzero(sp["hazard"] != 0)[0]
        ok, keep = ~np.isin(got[1], bad), ~np.isin(ids, bad)
        assert np.array_equal(got[0][ok], tiles[keep]) and np.array_equal(got[1][ok], ids[keep])
