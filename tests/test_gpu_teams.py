"""Compositing by whole workgroups against single waves: a view must come out
bit for bit the same alone (every tile by a workgroup), in a batch of medium size
(the long lists by workgroups) and in a large one (plain models: waves alone)."""
import numpy as np
import pytest
import torch

from gpu_helpers import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def r():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_18682_amd import renderer as R

    rr = R.Renderer(0)
    yield rr
    rr.close()


def _scene(n, logit, seed):
    """Gaussians in front of an identity camera, denser towards the axis."""
    rng = np.random.default_rng(seed)
    z = rng.uniform(2.0, 8.0, n)
    xy = rng.normal(0, 0.16, (2, n)) * z
    g = dict(means=np.stack([xy[0], xy[1], z]), log_scales=np.log(0.05 * z)[None] + rng.normal(0, 0.5, (3, n)),
             quats=rng.standard_normal((4, n)), opacity_logits=rng.normal(logit, 1.0, n), sh=rng.normal(0, 0.5, (1, 3, n)))
    g = {k: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).cuda() for k, v in g.items()}
    return dict(g, sh_degree=0)


def _cam(w, h, f):
    return dict(w2c=np.eye(3, 4), fx=f, fy=f, cx=w / 2, cy=h / 2, width=w, height=h)


# Lists of no entry, of less than a batch, of whole batches and one more, and of hundreds; faint Gaussians
# (no pixel stops) and opaque ones (all do); widths and heights that leave parts of tiles outside.
@pytest.mark.parametrize("tile", [(8, 8), (8, 16), (16, 8), (16, 16), (8, 32), (32, 8)])
@pytest.mark.parametrize("mip", [0, 2])
@pytest.mark.parametrize("n,logit,w,h", [(1, 0.0, 8, 8), (65, -2.0, 61, 47), (700, 3.0, 100, 75), (6000, -3.0, 131, 93)])
def test_teams_equal_waves(r, n, logit, w, h, mip, tile):
    say(f"case teams n {n} logit {logit} {w}x{h} mip {mip} tile {tile}")
    g = _scene(n, logit, n)
    cam = _cam(w, h, 0.9 * w)
    opts = dict(tile_w=tile[0], tile_h=tile[1], mip=mip)
    # other views of 1500 and 12000 tiles, which see few of the Gaussians
    def other(tiles):
        tw, th = 64, -(-tiles // 64)
        return dict(_cam(tw * tile[0], th * tile[1], 50.0), cx=-1e4)

    def first(cams):
        out = r.render(g, cams, opts)[0]
        return [out[k].cpu() for k in ("rgb", "final_T", "n_contrib")]

    alone = first([cam])
    for tiles in (1500, 12000):
        for a, b in zip(alone, first([cam, other(tiles)])):
            assert torch.equal(a, b)
    if n >= 6000:
        assert int(alone[2].max()) > 128


# Lists below a team's shortest, of one and of several batches to a wave; the last shape has 16 slots.
@pytest.mark.parametrize("tile", [(8, 8), (8, 16), (16, 16), (32, 32)])
@pytest.mark.parametrize("n,logit", [(40, 0.0), (300, -2.0), (2500, -4.0)])
def test_team_gradients(r, n, logit, tile):
    """Exact MIP gradients of a view alone (long lists by four waves together) and
    beside a view without upstream gradient whose instances raise the average
    work of a wave above every list (waves alone)."""
    say(f"case team gradients n {n} logit {logit} tile {tile}")
    from paper_2503_18682_amd import _lib as L

    g = _scene(n, logit, n)
    cam = _cam(101, 77, 90.0)
    opts = dict(tile_w=tile[0], tile_h=tile[1], mip=2)
    # the same Gaussians seen large, until the instances suffice
    reps = max(1, 3000 // n)
    wide = [dict(_cam(2000, 2000, 1800.0)) for _ in range(reps)]

    def grads(cams):
        dl = [torch.zeros(3, c["height"], c["width"], device="cuda") for c in cams]
        dl[0] = torch.rand(3, cam["height"], cam["width"], generator=torch.Generator().manual_seed(3)).cuda() - 0.4
        outs, (buf, ws) = r.render(g, cams, opts, flags=L.RGS_WS_BACKWARD, keep_workspace=True)
        return r.backward(g, cams, outs, dl, ws, opts), outs[0]

    a, out = grads([cam])
    b, _ = grads([cam] + wide)
    if n == 2500:
        assert int(out["n_contrib"].max()) > 256
    # T and the colour term pass up to 2500 roundings of 2^-24 in either order, and the terms of a
    # gradient may cancel to a tenth
    tol = 2 * 2500 * 2.0 ** -24 * 10
    for k in ("means", "log_scales", "quats", "opacity_logits", "sh"):
        top = float(a[k].abs().max())
        assert top > 0 and float((a[k] - b[k]).abs().max()) <= tol * top, k


# Frames of more tiles than all teams take, with lists that are split
@pytest.mark.parametrize("tile", [(8, 16), (16, 16), (8, 32)])
def test_alike_lists_equal_teams(r, tile):
    """Exact MIP with lists that are nearly alike (no teams) and beside a view of few, far longer lists (teams): the same
    bits."""
    from gpu_helpers import instance_lists, render_with_ws

    say(f"case alike lists tile {tile}")
    rng = np.random.default_rng(23)
    n, w, h = 40000, 701, 533
    z = rng.uniform(2.0, 8.0, n)
    xy = np.stack([rng.uniform(-0.6, 0.6, n), rng.uniform(-0.48, 0.48, n)]) * z
    g = dict(means=np.stack([xy[0], xy[1], z]), log_scales=np.log(0.02 * z)[None] + rng.normal(0, 0.3, (3, n)),
             quats=rng.standard_normal((4, n)), opacity_logits=rng.normal(-3.0, 0.5, n),
             sh=rng.normal(0, 0.5, (1, 3, n)))
    g = {k: np.ascontiguousarray(v, dtype=np.float32) for k, v in g.items()}
    g["sh_degree"] = 0
    cam, far = _cam(w, h, 0.9 * w), _cam(512, 512, 12.0)
    opts = dict(tile_w=tile[0], tile_h=tile[1], mip=2)

    def first(cams):
        outs, buf, _, lay, _ = render_with_ws(r, g, cams, opts)
        count = np.bincount(instance_lists(buf, lay)[0])
        # two workgroups of eight waves on a CU; lists of 128 and more count twice, unless the average work is larger
        waves = 16 * torch.cuda.get_device_properties(0).multi_processor_count
        split = count >= max(128, -(-int(count.sum()) // waves))
        return outs[0], count.max() * waves / (count.sum() + count[split].sum()), int(split.sum())

    alone, ratio, split = first([cam])
    assert ratio < 3 and split > 100
    beside, ratio, split = first([cam, far])
    assert ratio > 3 and split > 100
    for k in ("rgb", "final_T", "n_contrib"):
        assert np.array_equal(alone[k], beside[k])
