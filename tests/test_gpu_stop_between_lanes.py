"""The forward whose four lanes a pixel take eight list positions each: a pixel that
stops where one lane's positions end.  The next lane starts from T times the
product of the earlier lanes' (1 - alpha), a differently rounded product: it may
fall below 1e-4 where the sequence of products did not.  Gaussians on the optical
axis whose alphas are their opacities at the centre of the pixel they meet, with
opacities searched on the CPU (float32, the kernel's order) for that case.

Expected: the pixel keeps the T of the last blend (the FP32 rule, 1e-5, of the
product in FP64) and its count, and the adjoint, which recovers T by division from
it, the first Gaussian's weight (2e-5: forty divisions more)."""
import numpy as np
import pytest
import torch

import scenegen

f32 = np.float32
T_MIN = f32(1e-4)


def opacities(seed):
    """72 opacities: T * product of positions 32 .. 39 < 1e-4 <= the sequential product there."""
    rng = np.random.default_rng(seed)
    while True:
        a = rng.uniform(0.05, 0.13, 32).astype(f32)
        om = f32(1.0) - a
        prod = [np.multiply.reduce(om[8 * q:8 * q + 8], dtype=f32) for q in range(3)]
        T = (prod[0] * prod[1]) * prod[2]
        for x in om[24:]:
            T = T * x
        b = rng.uniform(0.4, 0.6, 8).astype(f32)
        head = T
        for x in f32(1.0) - b[:7]:
            head = head * x
        b[7] = f32(1.0) - T_MIN / head
        if not 0.05 < b[7] < 0.95:
            continue
        for _ in range(8):                        # a few neighbouring values of the last one
            P, S = f32(1.0), T
            for x in f32(1.0) - b:
                P, S = P * x, S * x
            if T * P < T_MIN <= S:
                return np.concatenate([a, b, np.full(32, 0.5, f32)])
            b[7] = np.nextafter(b[7], f32(0.0))


def test_search_finds_the_case():
    o = opacities(0).astype(np.float64)
    assert abs(np.prod(1 - o[:40]) / 1e-4 - 1) < 1e-6 and (o[40:] == 0.5).all()


@pytest.mark.gpu
@pytest.mark.parametrize("form,d,fdt", [("bf16", 32, "bf16"), ("bf16", 256, "bf16"), ("f32", 32, "f32")])
def test_stop_between_two_lanes(form, d, fdt):
    from paper_2505_19154_amd.raster import Gaussians, Rasterizer
    w = 17                                         # (the axis meets the centre of pixel 8, 8)
    cam = scenegen.look_at_camera((0, -4, 0), w, w)
    t = lambda a: torch.tensor(np.asarray(a, np.float32)).cuda()
    for seed in range(4):
        o = opacities(seed)
        n = len(o)
        means = np.zeros((n, 3))
        means[:, 1] = np.linspace(-1.0, 1.0, n)
        feat = torch.ones(n, d, device="cuda", dtype=torch.bfloat16 if fdt == "bf16" else torch.float32)
        g = Gaussians(t(means), t(np.full((n, 3), 0.3)), t(np.tile([1.0, 0, 0, 0], (n, 1))), t(o),
                      t(np.full((n, 1, 3), 0.5)), feat, 0)
        r = Rasterizer([cam], n, 0, d, feat_dtype=fdt, form=form)
        img = r.forward(g)
        pix = 8 * w + 8
        T64 = float(np.prod(1 - o[:40].astype(np.float64)))
        assert int(img.n_iter[pix]) == 40
        assert abs(float(img.T[pix]) / T64 - 1) <= 1e-5
        dC = torch.zeros(w * w, 3, device="cuda")
        dC[pix, 0] = 1.0
        got = float(r.render_bwd(g, img, dC)["sh"][0, 0, 0])
        assert abs(got / (float(o[0]) * 0.28209479177387814) - 1) <= 2e-5
