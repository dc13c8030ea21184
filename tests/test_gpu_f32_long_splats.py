"""The FP32-form adjoint of a splat's centre for long thin splats.  The conic's
row A dx + B dy nearly cancels along such a splat (its large part is q2 b with b
the distance from the long axis), so sums of dL/dpower dx and dL/dpower dy
multiplied by A and B afterwards show their rounding 3 to 10 times as large as
a sum of the per-pixel terms formed in the splat's own axes.

One Gaussian an image (T = 1, so dL/dpower = alpha rgb . dC), axes of about 60 and
1.5 pixels at eighteen angles.  Reference: FP64 from the record that the kernel
reads.  Measure: the error over the sum of the terms' sizes, root mean square over
the angles and both components.  Bound: twice that of a plain float32
evaluation (per-pixel terms, numpy's pairwise sum) of the same formula, the
factor for the spread between two orders of summation."""
import numpy as np
import pytest
import torch

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu

f32 = np.float32


def _terms(rec, w, h, t):
    """The terms of dL/d(u, v) in float type t (rgb . dC as one factor); FP64: no rounding."""
    r = rec.astype(t)
    x, y = np.meshgrid(np.arange(w) + 0.5, np.arange(h) + 0.5)
    dx, dy = (x.astype(t) - r[0]) - r[2], (y.astype(t) - r[1]) - r[3]
    ex, ey, q1, q2 = r[4], r[5], r[6], r[7]
    fma = lambda a, b, c: (np.float64(a) * np.float64(b) + np.float64(c)).astype(t)
    a, b = fma(ex, dx, ey * dy), fma(ex, dy, -(ey * dx))
    alpha = np.minimum(t(f32(0.99)), r[8] * np.exp2(fma(q1, a * a, q2 * (b * b))))
    if np.abs(alpha.astype(np.float64) * 255.0 - 1.0).min() < 5e-5:
        return None                       # (a pixel that float32 may blend or skip: 2e-5 is what alpha may be off)
    dp = np.where(alpha >= t(f32(1.0) / f32(255.0)), alpha * (r[9] + r[10] + r[11]), t(0))
    k = t(-2.0 * np.log(2.0))
    return [(k * dp * (q1 * a * ex - q2 * b * ey)).astype(t), (k * dp * (q1 * a * ey + q2 * b * ex)).astype(t)]


def test_centre_gradient_of_long_splats():
    from paper_2505_19154_amd.raster import Gaussians, Rasterizer
    w, h = 200, 190
    cam = scenegen.look_at_camera((0, -4, 0), w, h)
    rng = np.random.default_rng(12)
    gpu, plain = [], []
    t = lambda a: torch.tensor(np.asarray(a, np.float32)).cuda()
    for k in range(18):
        th = np.pi * (k + 0.37) / 18.0
        quat = [[np.cos(th / 2), 0.0, np.sin(th / 2), 0.0]]          # about the viewing axis
        g = Gaussians(t(rng.uniform(-0.05, 0.05, (1, 3))), t([[1.39, 0.032, 0.032]]), t(quat), t([0.8]),
                      t(rng.uniform(0.2, 1.0, (1, 1, 3))), None, 0)
        r = Rasterizer([cam], 1, 0, 0, form="f32")
        img = r.forward(g)
        r.render_bwd(g, img, torch.ones(w * h, 3, device="cuda"))
        torch.cuda.synchronize()
        rec = r.ws_view("rec", torch.float32, 12).cpu().numpy()
        row = r.ws_view("grad2d", torch.float32, 12).cpu().numpy().astype(np.float64)
        exact, single = _terms(rec, w, h, np.float64), _terms(rec, w, h, np.float32)
        if exact is None or single is None:
            continue
        for c in range(2):
            size = np.abs(exact[c]).sum()
            gpu.append(abs(row[c] - exact[c].sum()) / size)
            plain.append(abs(float(single[c].sum(dtype=f32)) - exact[c].sum()) / size)
    rms = lambda e: float(np.sqrt(np.mean(np.square(e))))
    print(f"[long splats] dL/d(u, v): kernel {rms(gpu):.2e}, per-pixel terms in float32 {rms(plain):.2e}", flush=True)
    assert len(gpu) >= 24 and rms(gpu) <= 2.0 * rms(plain)
