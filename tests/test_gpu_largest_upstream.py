"""Upstream feature adjoints near the largest float (3.40e38, above the largest
finite BF16 of 3.39e38): in the FP32 form with BF16 features of 256 channels and up,
dF enters the matrix unit as three BF16 terms whose sum is dF, also there.  Every
Gaussian has one channel that is not zero, of 2^-70: f . dF is then one product,
whose terms and their partial sums are exact whichever three terms the value is
split into, and finite.  So the gradients equal those of dF 2^-64, times 2^64, bit
for bit."""
import pytest
import torch

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [256, 264])
def test_largest_finite_upstream(d):
    from paper_2505_19154_amd.raster import Rasterizer
    g = scenegen.make_gaussians(150, 1.0, 0, d, seed=4, feat_dtype="bf16")
    cams = [scenegen.look_at_camera((0, -4, 0), 40, 24)]
    dg = U.device_gaussians(g)
    dg.feat = torch.zeros_like(dg.feat)
    dg.feat[torch.arange(150), torch.arange(150) * 7 % d] = 2.0 ** -70
    r = Rasterizer(cams, dg.n, 0, d, feat_dtype="bf16", form="f32")
    img = r.forward(dg)
    P = 40 * 24
    dC = torch.zeros(P, 3, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(1)
    dF = (torch.rand(P, d, device="cuda", generator=gen) - 0.5) * 2.0 ** 127
    big = torch.rand(P, d, device="cuda", generator=gen) < 0.01
    dF[big] = torch.finfo(torch.float32).max * torch.sign(dF[big])
    dF[0, :2] = torch.tensor([3.397e38, -3.401e38], device="cuda")
    got = {k: v.clone() for k, v in r.render_bwd(dg, img, dC, dF).items()}
    ref = r.render_bwd(dg, img, dC, dF * 2.0 ** -64)
    for k in ("means", "scales", "quats", "opacity"):
        assert torch.isfinite(got[k]).all() and got[k].abs().max() > 0
        assert torch.equal(got[k], ref[k] * 2.0 ** 64), k
