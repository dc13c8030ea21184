"""A Gaussian with an infinite colour component: the pixels that blend it hold an
infinity in that component, all others keep their bits (exact), in every shape of
the forward whose walk has no branch (0 * inf may not enter its sums) and in the
sequential one."""
import pytest
import torch

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,d,fdt,prim,shape", [
    ("bf16", 32, "bf16", "gaussian", None), ("bf16", 96, "bf16", "surfel", None), ("bf16", 128, "bf16", "gaussian", (128, 8)),
    ("bf16", 128, "bf16", "gaussian", (128, 16)), ("bf16", 256, "bf16", "gaussian", None), ("bf16", 256, "bf16", "surfel", None),
    ("f32", 64, "f32", "gaussian", None), ("f32", 256, "f32", "gaussian", None), ("f32", 16, "f32", "gaussian", None)])
def test_infinite_colour_stays_with_the_pixels_that_blend_it(form, d, fdt, prim, shape):
    from paper_2505_19154_amd.raster import Rasterizer
    n = 200
    g = scenegen.make_gaussians(n, 1.0, 1, d, seed=9, feat_dtype=fdt)
    cams = [scenegen.look_at_camera((0, -4, 0), 60, 44)]
    dg = U.device_gaussians(g)
    r = Rasterizer(cams, n, dg.sh_degree, d, feat_dtype=fdt, form=form, primitive=prim)
    if shape:
        r.set_tuning(shape[0], 32, shape[1])
    first = r.forward(dg)
    C0, T0, it0 = first.C.clone(), first.T.clone(), first.n_iter.clone()
    marked = {7: (0,), 50: (1, 2), 51: (1,), 199: (0, 1, 2)}
    want = C0.clone()
    keep = dg.feat
    for i, channels in marked.items():          # each marked Gaussian's weights, as a feature map
        dg.feat = torch.zeros_like(keep)
        dg.feat[i] = 1.0
        on = r.forward(dg).F[:, 0] > 0
        for c in channels:
            want[on, c] = float("inf")
    dg.feat = keep
    assert torch.isinf(want).any(0).all() and (torch.isinf(want).sum(0) < want.shape[0] // 2).all()
    for i, channels in marked.items():
        for c in channels:
            dg.sh[i, 0, c] = float("inf")
    img = r.forward(dg)
    assert torch.equal(img.C, want)
    assert torch.equal(img.T, T0) and torch.equal(img.n_iter, it0)
