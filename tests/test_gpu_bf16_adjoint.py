"""The BF16-form adjoint and fusion against the FP64 oracle where their tiling can
go wrong: one to four resident 32-channel slabs, 256 channels (the contraction
kernel and the walk apart), one and two slices above; lists whose first chunk
holds 1, 15, 16, 17 or 31 positions, one and two full pairs of chunks, one past
them; both primitives, with and without dF.  Tolerance: the BF16-form rule of
tests/gpu_util.py, as for the form's other tests."""
import numpy as np
import pytest

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _check(g, cams, vts, gpu, rule):
    ora = U.run_oracle(g, cams, vts, fusion=True, bin_rule=rule)
    keep = U.checkable(ora["gflags"])
    for k in ("means", "scales", "quats", "opacity", "sh"):
        ref = ora["grads"][k]
        m = keep.reshape((-1,) + (1,) * (ref.ndim - 1)) & np.ones(ref.shape, bool)
        mx, _ = U.elementwise(gpu["grads"][k].cpu().numpy(), ref, ora["grads_mag"][k], mask=m, amb=ora["grads_amb"][k],
                              rtol=U.RTOL_FORM["bf16"])
        print(f"[d={g['d']} {rule}] grad {k}: {mx:.3f}", flush=True)
        assert mx <= 1.0, k
    s = (gpu["acc"].sum + gpu["acc"].comp).cpu().numpy()
    m = keep[:, None] & np.ones(s.shape, bool)
    assert U.elementwise(s, ora["fsum"], ora["fsum_mag"], mask=m, amb=ora["fsum_amb"], rtol=U.RTOL_FORM["bf16"])[0] <= 1.0


@pytest.mark.parametrize("d,rule", [(32, "box"), (64, "surfel"), (96, "box"), (128, "surfel"), (256, "box"),
                                    (256, "surfel"), (384, "box"), (512, "surfel")])
def test_widths(d, rule):
    g = scenegen.make_gaussians(700, 1.2, 1, d, seed=60 + d, feat_dtype="bf16")
    if rule == "surfel":
        g["scales"] = (np.asarray(g["scales"]) * 3.0).astype(np.float32)
    cams = [scenegen.look_at_camera(p, w, h) for p, w, h in (((0, -4, 0), 50, 35), ((3, -2.5, 1.2), 33, 20))]
    vts = U.view_maps(cams, d, target_dtype="bf16")
    _check(g, cams, vts, U.run_gpu(g, cams, vts, fusion=True, form="bf16", bin_rule=rule), rule)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 49, 64])
def test_list_lengths(n):
    g = scenegen.make_gaussians(n, 0.3, 1, 32, seed=5, feat_dtype="bf16")
    g["scales"] = np.full((n, 3), 1.5, np.float32)
    g["opacity"] = np.full(n, 0.05, np.float32)
    cams = [scenegen.look_at_camera((0, -4, 0), 17, 16)]
    vts = U.view_maps(cams, 32, target_dtype="bf16")
    gpu = U.run_gpu(g, cams, vts, fusion=True, form="bf16")
    assert int(gpu["img"].n_iter.max()) == n
    _check(g, cams, vts, gpu, "box")
