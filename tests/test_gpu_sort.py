"""The binning at the sizes where its sorts change route: one workgroup sorts up
to 16384 keys of a segment (2, 8 or 16 keys a thread); above that tiles of 4096
keys, each workgroup adding up the digit counts of all; from 1.5M keys or 221
rows on tiles of 8192, with a scan of the counts for many rows.  The sorted
instances against numpy (exact): tile, depth and index order, ranges, ranks."""
import numpy as np
import pytest
import torch

import scenegen
from tests import gpu_util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,views,scale", [
    (1, 1, 1.0), (63, 2, 1.0), (2048, 1, 0.5), (2049, 2, 1.0), (8193, 1, 1.0), (16384, 2, 0.5), (16385, 2, 1.0),
    (40000, 3, 2.0), (300000, 1, 1.0), (120000, 16, 0.5), (1000001, 1, 0.5), (70000, 1, 40.0)])
def test_instances_are_sorted_by_tile_depth_and_index(n, views, scale):
    from paper_2505_19154_amd.raster import Rasterizer
    g = scenegen.make_gaussians(n, 2.0, 0, 0, seed=n % 97)
    g["scales"] = (np.asarray(g["scales"]) * scale).astype(np.float32)
    if n > 2:                                     # equal depths: index order
        g["means"] = np.asarray(g["means"]).copy()
        g["means"][1::2] = g["means"][0::2][: len(g["means"][1::2])]
    rng = np.random.default_rng(3)
    cams = [scenegen.look_at_camera(tuple(4.0 * d / np.linalg.norm(d)), 97 + 40 * i, 70 + 8 * i)
            for i, d in enumerate(rng.normal(size=(views, 3)))]
    dg = U.device_gaussians(g)
    r = Rasterizer(cams, n, 0, 0)
    r.prepare(dg)
    for _ in range(2):                            # (a second pass over the same buffers)
        r.project(dg)
        r.bin_sort()
    c = r.counters()
    assert not c.inst_overflow
    keys, gids = r.bin_keys(int(c.n_instances))
    keys, gids = keys.cpu().numpy().view(np.uint64), gids.cpu().numpy().astype(np.int64)
    total = n * views
    rect = r.ws_view("rect", torch.int32, 4 * total).cpu().numpy().reshape(views, n, 4)
    dk = r.ws_view("depth_key", torch.int32, total).cpu().numpy().view(np.uint32).reshape(views, n)
    ref_k, ref_g, t0 = [], [], 0
    for v, cam in enumerate(cams):
        tx, ty = -(-cam.width // 16), -(-cam.height // 16)
        x0, y0, x1, y1 = rect[v].T.astype(np.int64)
        on = (x0 <= x1) & (y0 <= y1)
        idx = np.nonzero(on)[0]
        wd, ht = (x1 - x0 + 1)[idx], (y1 - y0 + 1)[idx]
        rep = np.repeat(np.arange(idx.size), wd * ht)
        local = np.arange(rep.size) - np.repeat(np.cumsum(wd * ht) - wd * ht, wd * ht)
        tile = t0 + (y0[idx][rep] + local // wd[rep]) * tx + x0[idx][rep] + local % wd[rep]
        ref_k.append((tile.astype(np.uint64) << np.uint64(32)) | dk[v][idx][rep].astype(np.uint64))
        ref_g.append(idx[rep])
        t0 += tx * ty
    ref_k, ref_g = np.concatenate(ref_k), np.concatenate(ref_g)
    o = np.lexsort((ref_g, ref_k))
    assert c.n_instances == ref_k.size
    assert np.array_equal(keys, ref_k[o]) and np.array_equal(gids, ref_g[o])
    ranges = r.ws_view("ranges", torch.int32, 2 * t0).cpu().numpy().reshape(-1, 2)
    tiles = (ref_k[o] >> np.uint64(32)).astype(np.int64)
    first, last = np.searchsorted(tiles, np.arange(t0), "left"), np.searchsorted(tiles, np.arange(t0), "right")
    has = last > first
    assert np.array_equal(ranges[has, 0], first[has]) and np.array_equal(ranges[has, 1], last[has])
    assert not ranges[~has].any()
    binned = (rect[..., 0] <= rect[..., 2]) & (rect[..., 1] <= rect[..., 3])
    order = r.ws_view("order", torch.int32, total).cpu().numpy().reshape(views, n)
    rank = r.ws_view("rank_of", torch.int32, total).cpu().numpy().reshape(views, n)
    for v in range(views):                        # (ranks of Gaussians that some list holds)
        on = binned[v][order[v]]
        assert np.array_equal(rank[v][order[v]][on], np.arange(n)[on])
