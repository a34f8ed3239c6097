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
