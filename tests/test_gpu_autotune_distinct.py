"""Launch shapes that start the same kernels: the autotuner leaves the plan's own
fields where only one launch exists (the FP32 form's adjoint, its sequential
forward), whatever they are, instead of picking between equal timings."""
import pytest

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,fdt,rule", [(64, "bf16", "box"), (40, "f32", "box"), (64, "f32", "surfel")])
def test_autotune_keeps_fields_that_select_nothing(d, fdt, rule):
    from paper_2505_19154_amd.raster import Rasterizer
    g = scenegen.make_gaussians(400, 1.0, 0, d, seed=2, feat_dtype=fdt)
    cams = [scenegen.look_at_camera((0, -4, 0), 48, 40)]
    vts = U.view_maps(cams, d)
    dg = U.device_gaussians(g)
    dC, dF = U.concat(vts, "dC"), U.concat(vts, "dF")
    r = Rasterizer(cams, dg.n, 0, d, feat_dtype=fdt, form="f32", primitive="surfel" if rule == "surfel" else "gaussian")
    img = r.forward(dg)
    for shape in ((8, 16), (64, 32), (32, 16), (16, 32)):
        r.set_tuning(*shape)
        pick = r.autotune(dg, img, dC, dF, reps=1)
        assert (pick["fwd_slice"], pick["bwd_chunk"], pick["fwd_rows"], pick["schedule"]) == shape + (16, 0)
