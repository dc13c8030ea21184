"""The FP32-form adjoint and fusion (FP32 matrix contractions) against the FP64
oracle at the widths and sizes where their tiling can go wrong: feature widths
that fill no 16-channel block, that are not multiples of four (element loads),
one past a resident width, and above 256 channels (streamed slices); features
and upstream maps whose rows are not 16-byte aligned; lists of one position and
of one past a 32-position chunk.  Tolerance: the FP32 rule of tests/gpu_util.py
(rtol 1e-5 of the magnitude companion), as for the form's other widths."""
import numpy as np
import pytest
import torch

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _check(g, cams, vts, gpu, rule):
    ora = U.run_oracle(g, cams, vts, fusion=g["d"] > 0, bin_rule=rule)
    keep = U.checkable(ora["gflags"])
    for k in ("means", "scales", "quats", "opacity", "sh"):
        ref = ora["grads"][k]
        m = keep.reshape((-1,) + (1,) * (ref.ndim - 1)) & np.ones(ref.shape, bool)
        mx, _ = U.elementwise(gpu["grads"][k].cpu().numpy(), ref, ora["grads_mag"][k], mask=m, amb=ora["grads_amb"][k])
        print(f"[d={g['d']} {g['feat_dtype']} {rule}] grad {k}: {mx:.3f}", flush=True)
        assert mx <= 1.0, k
    if g["d"]:
        s = (gpu["acc"].sum + gpu["acc"].comp).cpu().numpy()
        w = (gpu["acc"].wsum + gpu["acc"].wcomp).cpu().numpy()
        m = keep[:, None] & np.ones(s.shape, bool)
        assert U.elementwise(s, ora["fsum"], ora["fsum_mag"], mask=m, amb=ora["fsum_amb"])[0] <= 1.0
        assert U.elementwise(w, ora["wsum"], ora["wsum"], mask=keep, amb=ora["wsum_amb"])[0] <= 1.0


@pytest.mark.parametrize("d,fdt,rule", [
    (0, "f32", "box"), (3, "f32", "box"), (17, "f32", "surfel"), (48, "bf16", "box"), (100, "f32", "box"),
    (129, "bf16", "box"), (256, "bf16", "surfel"), (257, "f32", "box"), (320, "bf16", "surfel"), (1024, "f32", "box")])
def test_adjoint_and_fusion_match_the_oracle(d, fdt, rule):
    g = scenegen.make_gaussians(700, 1.2, 1, d, seed=40 + d, feat_dtype=fdt)
    if rule == "surfel":
        g["scales"] = (np.asarray(g["scales"]) * 3.0).astype(np.float32)
    cams = [scenegen.look_at_camera(p, w, h) for p, w, h in (((0, -4, 0), 50, 35), ((3, -2.5, 1.2), 33, 20))]
    vts = U.view_maps(cams, d)
    gpu = U.run_gpu(g, cams, vts, fusion=d > 0, form="f32", bin_rule=rule)
    _check(g, cams, vts, gpu, rule)


@pytest.mark.parametrize("n", [1, 32, 33])
def test_short_lists(n):
    """n Gaussians that cover the whole image: lists of one position, one chunk, one position past it."""
    g = scenegen.make_gaussians(n, 0.3, 1, 20, seed=5)
    g["scales"] = np.full((n, 3), 1.5, np.float32)
    g["opacity"] = np.full(n, 0.05, np.float32)
    cams = [scenegen.look_at_camera((0, -4, 0), 17, 16)]
    vts = U.view_maps(cams, 20)
    gpu = U.run_gpu(g, cams, vts, fusion=True, form="f32")
    assert int(gpu["img"].n_iter.max()) == n
    _check(g, cams, vts, gpu, "box")


@pytest.mark.parametrize("fdt", ["f32", "bf16"])
def test_unaligned_features(fdt):
    """Features at an address aligned to their elements only: the same gradients bit for bit."""
    from paper_2505_19154_amd.raster import Gaussians, Rasterizer
    g = scenegen.make_gaussians(500, 1.0, 1, 36, seed=8, feat_dtype=fdt)
    cams = [scenegen.look_at_camera((0, -4, 0), 40, 24)]
    vts = U.view_maps(cams, 36)
    dg = U.device_gaussians(g)
    flat = torch.empty(dg.feat.numel() + 1, dtype=dg.feat.dtype, device="cuda")[1:]
    off = Gaussians(dg.means, dg.scales, dg.quats, dg.opacity, dg.sh, flat.view(dg.feat.shape).copy_(dg.feat), dg.sh_degree)
    r = Rasterizer(cams, dg.n, dg.sh_degree, dg.d, feat_dtype=fdt, form="f32")
    img = r.forward(dg)
    dC, dF, dT = (U.concat(vts, k) for k in ("dC", "dF", "dT"))
    a = {k: v.clone() for k, v in r.render_bwd(dg, img, dC, dF, dT).items()}
    b = r.render_bwd(off, img, dC, dF, dT)
    for k in a:
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("prim", ["gaussian", "surfel"])
def test_nonfinite_upstream_stays_with_the_gaussians_it_blends(prim):
    """An infinite dC in one pixel changes only Gaussians that blend there: every other gradient keeps its bits."""
    from paper_2505_19154_amd.raster import Rasterizer
    g = scenegen.make_gaussians(300, 1.0, 1, 8, seed=3)
    cams = [scenegen.look_at_camera((0, -4, 0), 40, 32)]
    vts = U.view_maps(cams, 8)
    dg = U.device_gaussians(g)
    r = Rasterizer(cams, dg.n, dg.sh_degree, dg.d, form="f32", primitive=prim)
    img = r.forward(dg)
    dC, dF, dT = (U.concat(vts, k) for k in ("dC", "dF", "dT"))
    a = {k: v.clone() for k, v in r.render_bwd(dg, img, dC, dF, dT).items()}
    pix = int(torch.where(img.T < 0.9, img.T, torch.zeros_like(img.T)).argmax())   # a pixel that blends few
    one = torch.zeros_like(dC)
    one[pix] = 1.0
    touched = r.render_bwd(dg, img, one, None, None)["opacity"].clone() != 0
    touched |= r.render_bwd(dg, img, one, None, None)["sh"].abs().flatten(1).amax(1) != 0
    assert 0 < int(touched.sum()) < dg.n // 2
    bad = dC.clone()
    bad[pix] = float("inf")
    b = r.render_bwd(dg, img, bad, dF, dT)
    for k in a:
        assert torch.equal(a[k][~touched], b[k][~touched]), k
    assert not torch.isfinite(b["sh"][touched]).all()
