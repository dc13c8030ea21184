"""Images of few tiles in the BF16 form, whose lists the fusion kernel and f . dF cut
among several workgroups: the gradient walk leaves T at every 128th position from
the list's end and the fusion takes up from there.  Lists one short of, equal to and
one past a segment, past the sixteen segments of one round, images of one tile, of
448 (the last cut ones) and of 450.  Against the FP64 oracle under the BF16 form's
rule; the gradients of a call without fusion, whose walk leaves no T, are the same
bits."""
import numpy as np
import pytest
import torch

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


def _scene(n, d, seed):
    """n faint Gaussians over the whole view of a camera at distance 4: every list holds all of them."""
    g = scenegen.make_gaussians(n, 0.5, 0, d, seed=seed, feat_dtype="bf16")
    g["scales"] = np.random.default_rng(seed).uniform(1.5, 3.0, (n, 3)).astype(np.float32)
    g["opacity"] = np.random.default_rng(seed + 1).uniform(0.0045, 0.0065, n).astype(np.float32)
    return g


@pytest.mark.parametrize("n,d,size,rule", [
    (127, 32, (16, 16), "box"), (128, 128, (16, 16), "box"), (129, 256, (33, 20), "box"), (257, 128, (16, 16), "surfel"),
    (2100, 32, (9, 16), "box"), (2100, 384, (7, 5), "surfel"), (300, 96, (40, 24), "surfel"), (200, 32, (448, 256), "box"),
    (200, 32, (16 * 18, 16 * 25), "box"), (40, 256, (16, 16), "box")])
def test_fusion_of_cut_lists(n, d, size, rule):
    g = _scene(n, d, n % 50 + d)
    cams = [scenegen.look_at_camera((0, -4, 0), *size)]
    vts = U.view_maps(cams, d, target_dtype="bf16")
    gpu = U.run_gpu(g, cams, vts, fusion=True, form="bf16", bin_rule=rule)
    ora = U.run_oracle(g, cams, vts, fusion=True, bin_rule=rule)
    rt = U.RTOL_FORM["bf16"]
    keep = U.checkable(ora["gflags"])
    s = (gpu["acc"].sum + gpu["acc"].comp).cpu().numpy()
    w = (gpu["acc"].wsum + gpu["acc"].wcomp).cpu().numpy()
    ms = U.elementwise(s, ora["fsum"], ora["fsum_mag"], rtol=rt, mask=keep[:, None].repeat(d, 1), amb=ora["fsum_amb"])[0]
    mw = U.elementwise(w, ora["wsum"], ora["wsum"], rtol=rt, mask=keep, amb=ora["wsum_amb"])[0]
    print(f"[long lists] n {n} d {d} {size} {rule}: list {int(gpu['img'].n_iter.max())}, sums {ms:.3f}, weights {mw:.3f}", flush=True)
    assert ms <= 1.0 and mw <= 1.0
    for k in ("means", "scales", "quats", "opacity", "sh"):
        ref = ora["grads"][k]
        m = keep.reshape((-1,) + (1,) * (ref.ndim - 1)) & np.ones(ref.shape, bool)
        assert U.elementwise(gpu["grads"][k].cpu().numpy(), ref, ora["grads_mag"][k], rtol=rt, mask=m, amb=ora["grads_amb"][k])[0] <= 1.0, k
    alone = gpu["r"].render_bwd(gpu["g"], gpu["img"], U.concat(vts, "dC"), U.concat(vts, "dF"), U.concat(vts, "dT"))
    for k, v in alone.items():
        assert torch.equal(v, gpu["grads"][k]), k
