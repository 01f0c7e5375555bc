"""GPU parity of the neighbourhood scan at the edges of its column strips,
row blocks and tiles: widths around the 14, 30 and 62 owned columns of a lane
group, heights around the 8 rows of a block, and regions large enough to be
cut into several tiles whose tables are merged, in the plane and in volumes.
Same measure and bars as the family's other GPU tests (1e-12 of the FP64
table: every sum is formed from exact integers in double)."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (nz, ny, nx of one region filling its image but for a ragged corner, alpha)
SHAPES = [(1, 1, 1, 0), (1, 7, 14, 0), (1, 8, 15, 1), (1, 9, 30, 0), (1, 17, 31, 0), (1, 16, 62, 2), (1, 15, 63, 0),
          (1, 70, 64, 0), (1, 33, 130, 0), (1, 2, 2500, 0), (1, 2500, 2, 0), (2, 7, 14, 0), (3, 9, 15, 1),
          (5, 25, 31, 0), (2, 64, 63, 0), (40, 8, 9, 0), (3, 3, 700, 0)]


@pytest.mark.parametrize("nz,ny,nx,alpha", SHAPES)
def test_scan_edges(nz, ny, nx, alpha):
    import torch
    from oracle import neighbourhood as nb
    from paper_2603_12016_amd import nyx
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(nz * 7919 + ny * 31 + nx)
    I = rng.integers(0, 900, (nz, ny, nx)).astype(np.uint16)
    L = np.ones((nz, ny, nx), np.uint32)
    if ny > 2 and nx > 2:
        L[:, : ny // 3, : nx // 4] = 0          # a notch: neighbours outside the region
        L[-1, -1, -1] = 2                       # another label in the corner
    # a plane next to a volume in one batch: the tables are laid out for the volume's 26 neighbours
    P = rng.integers(0, 900, (1, 50, 60)).astype(np.uint16)
    Q = np.ones((1, 50, 60), np.uint32)
    batch = [(I, L)] + ([(P, Q)] if nz > 1 else [])
    want = np.concatenate([nb.table(i, l, 16, alpha)[1] for i, l in batch])
    images = [(torch.from_numpy(i.view(np.int16)).to(dev), torch.from_numpy(l.view(np.int32)).to(dev)) for i, l in batch]
    rois, got = nyx.nyx_neighbourhood_features(nyx.nyx_create(0), images, 16, alpha, nyx.NYX_FP64)
    got = got.cpu().numpy()
    assert got.shape == want.shape
    assert np.array_equal(np.isnan(got), np.isnan(want))
    M = np.zeros(want.shape[1])
    M[[nb.NAMES.index("NGLDM_DCENT"), nb.NAMES.index("GLDM_DE")]] = 1.0
    ok = np.isnan(want) | (np.abs(got - want) <= 1e-12 * np.maximum(np.abs(want), M))
    assert ok.all(), (np.argwhere(~ok)[:4], got[~ok][:4], want[~ok][:4])
