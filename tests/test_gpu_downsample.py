"""Box downsampling: the factors with loops of their own, others, rows that
are no multiple of a wide load, and a source that is not aligned for one."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("factor", [1, 2, 3, 4, 6, 8, 16])
@pytest.mark.parametrize("planes,h,w,shift", [(1, 1, 1, 0), (3, 5, 7, 0), (2, 33, 65, 1), (3, 40, 300, 2)])
def test_downsample(factor, planes, h, w, shift):
    from paper_2503_18682_amd import renderer as R

    r = R.Renderer(0)
    gen = torch.Generator().manual_seed(factor * 100 + w)
    flat = torch.rand(planes * h * w * factor * factor + shift, generator=gen).cuda()
    img = flat[shift:].view(planes, h * factor, w * factor)
    want = img.double().view(planes, h, factor, w, factor).mean(dim=(2, 4))
    # factor^2 sums of values below 1, each rounded to 2^-24 of at most factor^2, then one product
    tol = (factor * factor + 2) * 2.0 ** -24
    assert float((r.downsample(img, factor).double() - want).abs().max()) <= tol * float(want.max())
    r.close()
