"""Exact MIP gradients where the four waves of a workgroup may share a list: behind
opaque stacks, where the transmittance underflows, and against the walk of a
single wave."""
import numpy as np
import pytest
import torch

from gpu_helpers import say

pytestmark = pytest.mark.gpu
KEYS = ("means", "log_scales", "quats", "opacity_logits", "sh")


@pytest.fixture(scope="module")
def r():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2503_18682_amd import renderer as R

    rr = R.Renderer(0)
    yield rr
    rr.close()


def _cam(w, h):
    return dict(w2c=np.eye(3, 4), fx=0.9 * w, fy=0.9 * w, cx=w / 2, cy=h / 2, width=w, height=h)


def _dev(g):
    g = {k: torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).cuda() for k, v in g.items()}
    return dict(g, sh_degree=0)


def _stack(n, seed):
    """Opaque Gaussians one behind the other over the left of the view, faint ones over all of it."""
    rng = np.random.default_rng(seed)
    faint = 40
    z = np.concatenate([rng.uniform(3.0, 8.0, n), rng.uniform(2.0, 9.0, faint)])
    x = np.concatenate([rng.normal(-0.3, 0.02, n), rng.uniform(-0.5, 0.5, faint)]) * z
    y = np.concatenate([rng.normal(0.0, 0.02, n), rng.uniform(-0.4, 0.4, faint)]) * z
    size = np.log(np.concatenate([0.15 * z[:n], 0.1 * z[n:]]))
    m = n + faint
    return _dev(dict(means=np.stack([x, y, z]), log_scales=size[None] + rng.normal(0, 0.1, (3, m)),
                     quats=rng.standard_normal((4, m)),
                     opacity_logits=np.concatenate([np.full(n, 9.0), np.full(faint, -2.0)]),
                     sh=rng.normal(0.3, 0.3, (1, 3, m))))


# Stacks of about a batch, and of several batches to a wave; alpha is clamped at alpha_max in their middle, so that
# a share of 20 records (10 with alpha_max 0.9999) takes the product of 1 / (1 - alpha) past the largest float32.
@pytest.mark.parametrize("views", [1, 3])
@pytest.mark.parametrize("n,alpha_max,tile", [(60, 0.9999, (8, 8)), (90, 0.99, (8, 16)), (200, 0.99, (16, 16)),
                                              (200, 0.9999, (32, 32)), (300, 0.99, (16, 8))])
def test_gradients_behind_opaque_stacks(r, n, alpha_max, tile, views):
    """t_eps = 0: pixels whose transmittance is 0 pass no gradient (as from a walk by one wave), all others
    that of a frame in which the deep pixels stop and have no upstream gradient."""
    from paper_2503_18682_amd import _lib as L

    say(f"case opaque stack n {n} alpha_max {alpha_max} tile {tile} views {views}")
    g = _stack(n, n)
    cams = [_cam(120 - 13 * v, 72 + 9 * v) for v in range(views)]
    base = dict(mip=2, alpha_max=alpha_max, tile_w=tile[0], tile_h=tile[1])

    def frame(t_eps):
        opts = dict(base, t_eps=t_eps)
        outs, (buf, ws) = r.render(g, cams, opts, flags=L.RGS_WS_BACKWARD, keep_workspace=True)
        return opts, outs, buf, ws

    zero, stop = frame(0.0), frame(1e-8)
    gen = torch.Generator().manual_seed(5)
    up = [torch.rand(3, c["height"], c["width"], generator=gen).cuda() - 0.4 for c in cams]
    T = [o["final_T"] for o in zero[1]]
    assert all(int((t == 0).sum()) > 100 and int((t > 1e-2).sum()) > 100 for t in T)
    clear = [t > 1e-6 for t in T]  # stopped in neither frame
    got = r.backward(g, cams, zero[1], [u * (c | (t == 0)) for u, c, t in zip(up, clear, T)], zero[3], zero[0])
    want = r.backward(g, cams, stop[1], [u * c for u, c in zip(up, clear)], stop[3], stop[0])
    # both the same sums over at most n + 40 records a pixel in another association, 2 roundings of 2^-24 a record, and
    # the terms of a gradient may cancel to a hundredth
    tol = 2 * (n + 40) * 2.0 ** -24 * 100
    for k in KEYS:
        top = float(want[k].abs().max())
        assert bool(torch.isfinite(got[k]).all()), k
        assert top > 0 and float((got[k] - want[k]).abs().max()) <= tol * top, k


def _lists(kind):
    """A view and Gaussians with: lists that are few, but long beside the average; lists alike; fewer lists than workgroups."""
    rng = np.random.default_rng(17)
    w, h, n, spread = {"few": (701, 533, 3000, 0.03), "alike": (701, 533, 40000, 0.6), "small": (131, 93, 9000, 0.5)}[kind]
    z = rng.uniform(2.0, 8.0, n)
    xy = (rng.normal(0.0, spread, (2, n)) if kind == "few" else rng.uniform(-spread, spread, (2, n))) * z
    g = _dev(dict(means=np.stack([xy[0], xy[1], z]), log_scales=np.log(0.03 * z)[None] + rng.normal(0, 0.3, (3, n)),
                  quats=rng.standard_normal((4, n)), opacity_logits=rng.normal(-4.5, 0.5, n),
                  sh=rng.uniform(-1.0, 1.0, (1, 3, n))))
    return g, _cam(w, h)


@pytest.mark.parametrize("tile", [(8, 8), (8, 16), (16, 16), (32, 32)])
@pytest.mark.parametrize("kind", ["few", "alike", "small"])
def test_shared_lists_equal_single_walk(r, kind, tile):
    """Gradients as the kernel deals the lists against those of a walk by one wave, which an entry of 1e-12 in the
    final transmittance of one pixel of each 8x8 block asks for; that pixel has no upstream gradient in either."""
    from paper_2503_18682_amd import _lib as L

    say(f"case shared lists {kind} tile {tile}")
    g, cam = _lists(kind)
    opts = dict(mip=2, tile_w=tile[0], tile_h=tile[1])
    outs, (buf, ws) = r.render(g, [cam], opts, flags=L.RGS_WS_BACKWARD, keep_workspace=True)
    T, n = outs[0]["final_T"], int(outs[0]["n_contrib"].max())
    assert float(T.min()) > 1e-4 and n > 192
    up = 0.5 + 0.5 * torch.rand(3, cam["height"], cam["width"], generator=torch.Generator().manual_seed(3)).cuda()
    up[:, ::8, ::8] = 0.0
    a = r.backward(g, [cam], outs, [up], ws, opts)
    T[::8, ::8] = 1e-12
    b = r.backward(g, [cam], outs, [up], ws, opts)
    # The same terms, all positive in a colour's gradient, with up to n roundings of 2^-24 in T and in the
    # colour behind, in another association, and in another order of the up to 250 partial sums of a record
    tol = 2 * (n + 250) * 2.0 ** -24
    ca, cb = a["sh"][0], b["sh"][0]
    assert bool((cb >= 0).all()) and float(cb.max()) > 0
    assert float(((ca - cb).abs() - tol * cb).max()) <= 0
    # dL/d(logit) sums a (T rgd - S / (1 - a)), each part at most a T (largest colour) (sum of the upstream gradient)
    most = 2 * tol * (0.5 + 0.2820948) * (cb / 0.2820948).sum(0)
    assert float(((a["opacity_logits"] - b["opacity_logits"]).abs() - most).max()) <= 0
    for k in KEYS:
        top = float(b[k].abs().max())
        assert top > 0 and float((a[k] - b[k]).abs().max()) <= 20 * tol * top, k
