"""BUSYNESS where its denominator sum |i p_i - j p_j| vanishes although several
levels are present (i n_i alike for all of them): 0, exactly, as for a flat
texture; and beside it, one voxel off that balance, the quotient of the exact
sums.  Rows of k voxels of the top level and bins k - extra of the lowest."""
from __future__ import annotations

from fractions import Fraction

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bins", [2, 3, 7, 11, 50])
@pytest.mark.parametrize("fp64", [True, False])
def test_vanishing_denominator(bins, fp64):
    import torch
    from oracle import neighbourhood as nb
    from paper_2603_12016_amd import nyx
    rows = [(k, bins * k - extra) for k in range(1, 31) for extra in (0, 1)]
    L = np.zeros((len(rows) * 2, (bins + 1) * 30), np.uint32)
    I = np.zeros(L.shape, np.uint16)
    want = []
    for r, (top, low) in enumerate(rows):
        L[2 * r, :top + low] = r + 1
        I[2 * r, :top], I[2 * r, top:top + low] = 900, 100
        # in a row, only the two voxels at the border have a neighbour of the other level
        n, N = {1: low, bins: top}, top + low
        s = {1: Fraction(bins - 1, 2 if low > 1 else 1), bins: Fraction(bins - 1, 2 if top > 1 else 1)}
        ps = sum(Fraction(n[i], N) * s[i] for i in n)
        den = 2 * abs(Fraction(low, N) - bins * Fraction(top, N))
        want.append(float(ps / den) if den else 0.0)
    images = [(torch.from_numpy(I.view(np.int16)).cuda(), torch.from_numpy(L.view(np.int32)).cuda())]
    torch.cuda.synchronize()
    _, got = nyx.nyx_neighbourhood_features(nyx.nyx_create(0), images, bins, 0, nyx.NYX_FP64 if fp64 else nyx.NYX_FP32)
    got = got.cpu().numpy().astype(np.float64)[:, nb.NAMES.index("NGTDM_BUSYNESS")]
    want = np.array(want)
    assert (got[want == 0.0] == 0.0).all(), got[want == 0.0]
    np.testing.assert_allclose(got, want, rtol=1e-14 if fp64 else 1e-7, atol=0)
