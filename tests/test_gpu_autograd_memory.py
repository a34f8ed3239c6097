"""A differentiable render gives its workspace back with its last reference."""
import gc

import pytest
import torch

pytestmark = pytest.mark.gpu


def test_workspace_is_released_without_a_collection():
    from paper_2503_18682_amd import renderer as R
    import numpy as np

    r = R.Renderer(0)
    n = 500
    gen = torch.Generator().manual_seed(2)
    g = dict(means=torch.randn(3, n, generator=gen), log_scales=torch.full((3, n), -3.0),
             quats=torch.randn(4, n, generator=gen), opacity_logits=torch.zeros(n), sh=torch.rand(1, 3, n, generator=gen))
    g = {k: t.cuda().requires_grad_(True) for k, t in g.items()}
    cam = dict(w2c=np.array([[1.0, 0, 0, 0], [0, 1, 0, 0], [0, 0, 1, 4]]), fx=80.0, fy=80.0, cx=48.0, cy=32.0, width=96,
               height=64)

    def step(keep_graph):
        img, = R.render(r, dict(g, sh_degree=0), [cam])
        loss = (img ** 2).sum()
        if keep_graph:
            torch.autograd.grad(loss, list(g.values()))
        return float(loss.detach())

    step(True)
    gc.collect()
    gc.disable()
    try:
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated()
        for keep in (True, False, True):
            step(keep)
        torch.cuda.synchronize()
        assert torch.cuda.memory_allocated() == before
    finally:
        gc.enable()
    r.close()
