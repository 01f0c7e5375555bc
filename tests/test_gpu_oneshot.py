"""One-shot calls on one context, one after another: the two routes of ROI
discovery (descriptors sized by the label table, or counted first when the
label values are many) give the same tables; more ROIs than the binding made
room for; an error between two calls; and a stream of the caller's own.
Whole numbers are equal, FP64 tables within 1e-12 (double sums whose order may
follow the order of atomics)."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _images(stride):
    """Six blocks labelled stride, 2 stride, ...; with stride 30000 the label
    table has 180001 entries, more than discovery sizes descriptors by."""
    import torch
    rng = np.random.default_rng(4)
    L = np.zeros((450, 450), np.uint32)
    for k, (y, x, h, w) in enumerate([(3, 5, 20, 31), (40, 0, 64, 90), (120, 100, 7, 200), (200, 40, 90, 90),
                                      (300, 300, 1, 1), (330, 20, 110, 400)]):
        L[y:y + h, x:x + w] = (k + 1) * stride
    I = rng.integers(0, 5000, L.shape).astype(np.uint16)
    return [(torch.from_numpy(I.view(np.int16)).cuda(), torch.from_numpy(L.view(np.int32)).cuda())]


def _all(nyx, ctx, images, stream=None):
    offs = nyx.nyx_offsets_default(2, 1)
    out = []
    for rois, table in (nyx.nyx_extract_batch(ctx, images, 32, offs, nyx.NYX_FP64, mode="dense-scan", stream=stream),
                        nyx.nyx_intensity_features(ctx, images, 32, nyx.NYX_FP64, stream=stream),
                        nyx.nyx_neighbourhood_features(ctx, images, 32, 0, nyx.NYX_FP64, stream=stream)):
        assert rois.label.shape[0] == rois.n_rois == table.shape[0]
        out.append((table.cpu().numpy(), rois.n_vox.cpu().numpy(), rois.bbox.cpu().numpy()))
    rois, bins = nyx.nyx_bin_rois(ctx, images, 32, want_bins=True, stream=stream)
    g = nyx.nyx_glcm_accumulate(ctx, images, rois, 32, offs, stream=stream)
    out.append((bins.cpu().numpy(), g.keys.cpu().numpy(), g.counts.cpu().numpy()))
    return out


def _same(a, b):
    for x, y in zip(a, b):
        for u, v in zip(x, y):
            assert u.shape == v.shape and u.dtype == v.dtype
            if u.dtype.kind == "f":
                np.testing.assert_allclose(u, v, rtol=1e-12, atol=0)
            else:
                assert np.array_equal(u, v)


def test_discovery_routes_and_recovery():
    import torch
    from paper_2603_12016_amd import nyx
    ctx = nyx.nyx_create(0)
    want = _all(nyx, ctx, _images(1))
    _same(want, _all(nyx, ctx, _images(30000)))
    with pytest.raises(nyx.NyxError) as e:
        nyx.nyx_intensity_features(ctx, _images(1), 32, capacity=2)
    assert e.value.status == nyx.NYX_ERR_CAPACITY
    side = torch.cuda.Stream()
    images = _images(1)
    torch.cuda.synchronize()
    _same(want, _all(nyx, ctx, images, stream=side))


def test_more_rois_than_room_was_made_for():
    import torch
    from paper_2603_12016_amd import nyx
    ctx = nyx.nyx_create(0)
    n = 40 * 50
    L = (torch.arange(40 * 50, dtype=torch.int32, device="cuda") + 1).reshape(40, 50)
    L = L.repeat_interleave(3, 0).repeat_interleave(3, 1).contiguous()    # 2000 ROIs of 3 x 3 in 18000 voxels
    I = (torch.arange(L.numel(), dtype=torch.int32, device="cuda") % 977).to(torch.int16).reshape(L.shape)
    assert nyx._guess_rows([(I, L)], 37 * 4) < n
    rois, table = nyx.nyx_intensity_features(ctx, [(I, L)], 8)
    assert rois.n_rois == n and table.shape == (n, 37)
    mean = I.reshape(40, 3, 50, 3).permute(0, 2, 1, 3).reshape(n, 9).double().mean(1).float()
    assert torch.equal(table[:, 0], mean)
    rois, table = nyx.nyx_extract_batch(ctx, [(I, L)], 8, nyx.nyx_offsets_default(2, 1))
    assert rois.n_rois == n and table.shape == (n, 5, 30)
