"""What the autograd function keeps of a pass.

Backward needs T and n_iter of its forward; the images that forward returned
must go when the caller drops them, by reference counts alone: a loop that makes
few Python objects a pass runs the cycle collector so rarely that it would fill
the device with old feature maps first.  A stand-in for the rasterizer returns
images whose memory is watched.
"""
import gc
import weakref

import numpy as np
import pytest
import torch

from paper_2505_19154_amd import autograd
from paper_2505_19154_amd.raster import Image

N, P, D = 5, 12, 4


class _Watched(np.ndarray):
    """ndarray that takes weak references: the memory behind a tensor."""


class _Rasterizer:
    def __init__(self, d):
        self.generation = 0
        self.d = d
        self.images = []

    def _tensor(self, *shape):
        a = np.zeros(shape, np.float32).view(_Watched)
        t = torch.from_numpy(a)
        self.images.append(weakref.ref(a))
        return t

    def forward(self, g):
        self.generation += 1
        F = self._tensor(P, self.d) if self.d else None
        return Image(self._tensor(P, 3), F, self._tensor(P), torch.zeros(P, dtype=torch.int32))

    def render_bwd(self, g, img, dC, dF, dT):
        assert img.C.shape == dC.shape and (img.F is None) == (dF is None)
        return {k: torch.ones_like(getattr(g, k)) for k in ("means", "scales", "quats", "opacity", "sh")}


def _leaves():
    return [torch.zeros(N, w, requires_grad=True) if w else torch.zeros(N, requires_grad=True) for w in (3, 3, 4, 0, 3)]


@pytest.mark.parametrize("d", [0, D])
@pytest.mark.parametrize("backward", [False, True])
def test_images_go_with_the_callers_references(d, backward):
    leaves, r = _leaves(), _Rasterizer(d)
    feat = torch.zeros(N, d) if d else None
    gc.collect()
    gc.disable()
    try:
        C, F, T, n_iter = autograd.rasterize(r, *leaves, feat, 0)
        assert C.requires_grad and all(ref() is not None for ref in r.images)
        if backward:
            outs, ups = ([C, F], [torch.ones_like(C), torch.ones_like(F)]) if d else ([C], [torch.ones_like(C)])
            grads = torch.autograd.grad(outs, leaves, ups)
            assert all(torch.equal(x, torch.ones_like(y)) for x, y in zip(grads, leaves))
            del outs, ups, grads
        del C, F, T, n_iter
        left = sum(ref() is not None for ref in r.images)
    finally:
        gc.enable()
    assert left == 0
