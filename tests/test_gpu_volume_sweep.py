"""GPU parity of the 3D row sweep: exact counts against a numpy enumeration of
the voxel pairs at the edges of its strips (14, 30 and 62 owned columns), row
blocks (8 rows) and planes, for whole, partial, reordered and sign-flipped
sets of the 13 distance-1 offsets, sets it hands to the general path (a class
twice, a longer distance), planes next to volumes, and features in every
accumulation mode against those of the exact counts."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FULL = [(0, 0, 1), (0, 1, 0), (1, 0, 0), (0, 1, 1), (0, 1, -1), (1, 0, 1), (1, 0, -1), (1, 1, 0), (1, -1, 0),
        (1, 1, 1), (1, 1, -1), (1, -1, 1), (1, -1, -1)]
FLIPPED = [tuple(-v for v in o) for o in FULL[::-1]]
SETS = {"full": FULL, "flipped": FLIPPED, "plane": FULL[:2] + [(0, -1, 1)], "up": [(-1, 0, 0), (1, 1, 1)],
        "twice": [(0, 0, 1), (0, 0, -1), (1, 0, 0)], "far": [(0, 0, 2), (1, 0, 0), (1, 1, 1)]}
SHAPES = [(2, 7, 14), (3, 8, 15), (2, 9, 30), (4, 17, 31), (2, 16, 62), (3, 15, 63), (1, 24, 130), (6, 1, 64), (9, 33, 1),
          (30, 20, 20)]


def _case(shape):
    rng = np.random.default_rng(sum(shape))
    I = rng.integers(0, 700, shape).astype(np.uint16)
    L = np.ones(shape, np.uint32)
    L[rng.random(shape) < 0.1] = 0
    L[-1, : shape[1] // 2, shape[2] // 2:] = 5
    L.flat[0] = 1
    return I, L


def _counts(I, L, lab, off, ng):
    m = L == lab
    lo, hi = int(I[m].min()), int(I[m].max())
    lv = np.minimum(1 + ng * (I.astype(np.int64) - lo) // max(hi - lo, 1), ng)
    a = tuple(slice(max(-d, 0), n - max(d, 0)) for d, n in zip(off, I.shape))
    b = tuple(slice(max(d, 0), n - max(-d, 0)) for d, n in zip(off, I.shape))
    C = np.zeros((ng, ng), np.int64)
    if all(abs(d) < n for d, n in zip(off, I.shape)):
        both = m[a] & m[b]
        i, j = lv[a][both] - 1, lv[b][both] - 1
        np.add.at(C, (np.minimum(i, j), np.maximum(i, j)), 1)
    return C


def _device(pairs):
    import torch
    return [(torch.from_numpy(i.view(np.int16)).cuda(), torch.from_numpy(l.view(np.int32)).cuda()) for i, l in pairs]


@pytest.mark.parametrize("name", list(SETS))
@pytest.mark.parametrize("shape", SHAPES)
def test_counts_exact(name, shape):
    from paper_2603_12016_amd import nyx
    ng, offs = 16, SETS[name]
    pairs = [_case(shape), _case((2, 5, 9))]      # (the first may be a plane: one volume in the batch)
    ctx, images = nyx.nyx_create(0), _device(pairs)
    rois, _ = nyx.nyx_bin_rois(ctx, images, ng)
    g = nyx.nyx_glcm_accumulate(ctx, images, rois, ng, offs)
    key, cnt = g.keys.cpu().numpy().view(np.uint64), g.counts.cpu().numpy()
    got = np.zeros((rois.n_rois, len(offs), ng, ng), np.int64)
    f = [(key >> np.uint64(s)).astype(np.int64) for s in (38, 32, 16, 0)]
    got[f[0], f[1] & 63, f[2] & 0xFFFF, f[3] & 0xFFFF] = cnt
    row = 0
    for I, L in pairs:
        for lab in np.unique(L[L > 0]):
            for k, off in enumerate(offs):
                assert np.array_equal(got[row, k], _counts(I, L, lab, off, ng)), (lab, off)
            row += 1
    assert row == rois.n_rois


@pytest.mark.parametrize("mode,bins", [("auto", 64), ("dense16-scan", 16), ("dense-scan", 16), ("dense-list", 16),
                                       ("auto", 700)])
@pytest.mark.parametrize("name", ["full", "up"])
def test_features_of_the_counts(mode, bins, name):
    """Plans of every mode, split and unsplit regions, against the features of
    the exact counts (both FP64: 1e-12 of each feature's own magnitude, and of
    the column's for the signed ones, is 1e-9 of the column's largest value
    with room to spare)."""
    import torch
    from paper_2603_12016_amd import nyx
    pairs, offs = [_case((30, 20, 20)), _case((5, 9, 31)), _case((1, 12, 40))], SETS[name]
    ctx, images = nyx.nyx_create(0), _device(pairs)
    torch.cuda.synchronize()
    rois, _ = nyx.nyx_bin_rois(ctx, images, bins)
    want = nyx.nyx_glcm_features(ctx, nyx.nyx_glcm_accumulate(ctx, images, rois, bins, offs), nyx.NYX_FP64).cpu().numpy()
    plan = nyx.nyx_plan_create(ctx, images, bins, offs, nyx.NYX_FP64, mode=mode)
    table = nyx.new_table(plan, len(offs), nyx.NYX_FP64)
    for _ in range(2):
        nyx.nyx_plan_execute(plan, table)
    nyx.nyx_plan_check(plan)
    got = table.cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(want))
    top = np.nanmax(np.abs(want).reshape(-1, 30), axis=0)
    err = np.nan_to_num(np.abs(got - want)) / np.maximum(top, 1e-30)
    assert err.max() <= 1e-9, np.unravel_index(err.argmax(), err.shape)
