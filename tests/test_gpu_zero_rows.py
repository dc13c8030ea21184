"""The rows of the screen-space adjoints that no walk reached: the visit staging
clears all rows in order (by workgroups of its own where tiles are few) and the
reduction writes only those with visits.  Rows left from an earlier pass (NaN
here) may not show: zero where there is no visit, finite elsewhere, and the
gradients the same bits as those of a first pass (exact)."""
import pytest
import torch

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,views,size,prim", [
    (1, 1, (16, 16), "gaussian"), (300, 3, (50, 35), "gaussian"), (257, 2, (33, 20), "surfel"), (60000, 1, (17, 9), "gaussian")])
def test_rows_without_visits_are_zero(n, views, size, prim):
    from paper_2505_19154_amd.raster import Rasterizer
    g = scenegen.make_gaussians(n, 2.0, 0, 32, seed=n % 89, feat_dtype="bf16")
    cams = [scenegen.look_at_camera(p, *size) for p in ((0, -4, 0), (3, -2.5, 1.2), (-3, 2, 0))[:views]]
    r = Rasterizer(cams, n, 0, 32, feat_dtype="bf16", form="f32", primitive=prim)
    dg = U.device_gaussians(g)
    gw = 16 if prim == "surfel" else 12
    gen = torch.Generator(device="cuda").manual_seed(1)
    dC = torch.rand(r.n_pixels, 3, device="cuda", generator=gen)
    dF = torch.rand(r.n_pixels, 32, device="cuda", generator=gen)
    img = r.forward(dg)
    rows = r.ws_view("grad2d", torch.float32, n * views * gw)
    first = {k: v.clone() for k, v in r.render_bwd(dg, img, dC, dF).items()}
    rows.fill_(float("nan"))
    again = r.render_bwd(dg, img, dC, dF)
    rows = rows.view(views, n, gw).cpu()
    seg = r.ws_view("vseg", torch.int32, 2 * n * views).view(views, n, 2).cpu()
    order = r.ws_view("order", torch.int32, n * views).view(views, n).cpu().long()
    for v in range(views):
        bare = order[v][seg[v, :, 0] == seg[v, :, 1]]
        assert (rows[v][bare] == 0).all()
    assert torch.isfinite(rows).all()
    for k in first:
        assert torch.equal(first[k], again[k]), k
