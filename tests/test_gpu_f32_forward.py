"""The FP32-form forward (sequential walk, FP32 matrix contraction) against the
FP64 oracle at the widths and sizes where its tiling can go wrong: widths that
fill no 16-channel block or are not multiples of four, more than one
128-channel slice, lists of one position and of one past a chunk.  Tolerance:
the FP32 rule of tests/gpu_util.py, n_iter exactly where no decision is near
its threshold."""
import numpy as np
import pytest
import torch

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,fdt,rule", [
    (700, 0, "f32", "box"), (700, 3, "f32", "box"), (700, 16, "bf16", "surfel"), (700, 17, "f32", "surfel"),
    (700, 48, "bf16", "box"), (700, 100, "f32", "box"), (500, 129, "bf16", "box"), (500, 256, "bf16", "box"),
    (300, 272, "bf16", "surfel"), (1, 20, "f32", "box"), (32, 20, "f32", "box"), (33, 20, "f32", "box")])
def test_forward_matches_the_oracle(n, d, fdt, rule):
    g = scenegen.make_gaussians(n, 1.2 if n > 100 else 0.3, 1, d, seed=60 + d, feat_dtype=fdt)
    if rule == "surfel":
        g["scales"] = (np.asarray(g["scales"]) * 3.0).astype(np.float32)
    if n < 100:
        g["scales"] = np.full((n, 3), 1.5, np.float32)
    cams = [scenegen.look_at_camera(p, w, h) for p, w, h in (((0, -4, 0), 50, 35), ((3, -2.5, 1.2), 33, 20))]
    gpu = U.run_gpu(g, cams, form="f32", bin_rule=rule)
    ora = U.run_oracle(g, cams, U.view_maps(cams, d), bin_rule=rule)
    cat = lambda k: np.concatenate([v[k] for v in ora["views"]])
    ok = (cat("flags") & 1) == 0
    img = gpu["img"]
    assert np.array_equal(img.n_iter.cpu().numpy().astype(np.int64)[ok], cat("niter")[ok])
    assert U.elementwise(img.C.cpu().numpy(), cat("C"), cat("Cmag"), mask=ok[:, None].repeat(3, 1), amb=cat("Cden"))[0] <= 1.0
    assert U.elementwise(img.T.cpu().numpy(), cat("T"), cat("T"), mask=ok, amb=cat("Tden"))[0] <= 1.0
    if d:
        assert U.elementwise(img.F.cpu().numpy(), cat("F"), cat("Fmag"), mask=ok[:, None].repeat(d, 1),
                             amb=cat("Fden"))[0] <= 1.0


@pytest.mark.parametrize("fdt", ["f32", "bf16"])
def test_nonfinite_features_stay_with_the_pixels_that_blend_them(fdt):
    """inf, -inf and NaN in a few Gaussians' features: the pixels that blend none
    of them keep their bits, the others hold what the sum of their terms gives."""
    from paper_2505_19154_amd.raster import Rasterizer
    g = scenegen.make_gaussians(200, 1.0, 1, 16, seed=9, feat_dtype=fdt)
    cams = [scenegen.look_at_camera((0, -4, 0), 60, 44)]
    dg = U.device_gaussians(g)
    r = Rasterizer(cams, dg.n, dg.sh_degree, dg.d, feat_dtype=fdt, form="f32")
    F0 = r.forward(dg).F.clone()
    marked = torch.zeros_like(dg.feat)
    bad = {5: float("inf"), 40: float("-inf"), 41: float("inf"), 90: float("nan")}
    weights = {}
    for i in bad:                       # each marked Gaussian's weight map
        marked.zero_()
        marked[i] = 1.0
        keep, dg.feat = dg.feat, marked
        weights[i] = r.render_fwd(dg).F[:, 0].clone()
        dg.feat = keep
    feat = dg.feat.clone()
    for i, x in bad.items():
        feat[i, i % 16] = x
    dg.feat = feat
    F = r.render_fwd(dg).F
    want = F0.clone()
    for i, x in bad.items():
        want[:, i % 16] += torch.where(weights[i] > 0, torch.full_like(weights[i], x), torch.zeros_like(weights[i]))
    assert torch.isfinite(want).all(1).any() and not torch.isfinite(want).all()
    same = torch.isfinite(want)
    assert torch.equal(torch.isnan(F), torch.isnan(want)) and torch.equal(F[torch.isinf(want)], want[torch.isinf(want)])
    untouched = torch.stack([w == 0 for w in weights.values()]).all(0)
    assert torch.equal(F[untouched], F0[untouched]) and torch.isfinite(F[same]).all()
