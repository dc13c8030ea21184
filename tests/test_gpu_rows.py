"""Row kernels: densification's copies of per-Gaussian rows and the fusion
finalisation, at row sizes that take each access width (16, 4 and 1 bytes; rows
longer than a workgroup; rows that fill no power of two of lanes).  Copies are
compared bit for bit, finalised features with the same float32 operations in
torch (one IEEE operation each), bit for bit."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,shape,dtype,shift", [
    (1, (3,), torch.uint8, 0), (63, (7,), torch.uint8, 0), (64, (1,), torch.float32, 0), (65, (19,), torch.bfloat16, 0),
    (130, (20,), torch.float32, 0), (130, (20,), torch.float32, 1), (200, (256,), torch.bfloat16, 0),
    (5, (4099,), torch.float32, 0), (3, (5000,), torch.uint8, 0)])
def test_densify_carries_rows(n, shape, dtype, shift):
    from paper_2505_19154_amd import train as T
    gen = torch.Generator(device="cuda").manual_seed(n)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    p = T.activate(T.Params(r(n, 3), r(n, 3) - 3.0, r(n, 4), 3 * r(n), r(n, 4, 3)))
    m = T.Params(*[r(*getattr(p, k).shape) for k in T.GROUPS])
    count = torch.ones(n, dtype=torch.int32, device="cuda")
    gsum = r(n).abs() * 3e-4
    flat = torch.randint(0, 255, (n * int(np.prod(shape)) + shift,), generator=gen, device="cuda").to(dtype)[shift:]
    rows = flat.view((n,) + shape)
    out, om, _, (got,) = T.densify(p, m, m, gsum, count, r(n, 2, 3), 2e-4, -3.0, -2.0, extra_rows=(rows,))
    hot, kept = gsum >= 2e-4, p.logit_opacity >= -2.0
    split = hot & (p.log_scales.amax(1) > -3.0)
    first, extra = torch.nonzero(kept)[:, 0], torch.nonzero(kept & hot)[:, 0]
    src = torch.cat([first, extra])
    assert torch.equal(got, rows[src]) and torch.equal(out.sh, p.sh[src]) and torch.equal(out.quats, p.quats[src])
    old = torch.cat([~split[first], torch.zeros_like(extra, dtype=torch.bool)])
    for k in T.GROUPS:
        want = getattr(m, k)[src] * old.view(-1, *[1] * (getattr(m, k).dim() - 1))
        assert torch.equal(getattr(om, k), want), k


@pytest.mark.parametrize("n,d", [(1, 4), (300, 3), (300, 20), (77, 64), (50, 260), (9, 512), (3, 1024)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_fuse_finalize_rows(n, d, dtype):
    from paper_2505_19154_amd.raster import FusionAcc, fuse_finalize
    gen = torch.Generator(device="cuda").manual_seed(d)
    r = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    w = torch.where(r(n) > 0.3, r(n).abs(), torch.zeros(n, device="cuda"))
    acc = FusionAcc(r(n, d), 1e-7 * r(n, d), w, 1e-8 * w)
    feat = r(n, d).to(dtype)
    W = acc.wsum + acc.wcomp
    fused = ((acc.sum + acc.comp) / W[:, None]).to(dtype)
    for feat_in in (feat, None):
        want = torch.where(W[:, None] > 0, fused, feat if feat_in is not None else torch.zeros_like(feat))
        assert torch.equal(fuse_finalize(acc, feat_in, dtype), want)
