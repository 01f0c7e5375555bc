"""A plan's replays: the graph of one branch, the one of two that takes its
place where the outputs come back, and changes of the outputs between them (two
tables in turn, a per-ROI pass and a profile into others) write the same rows
into the table that was passed, and into that one only."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bins", [256, 600])
def test_outputs_between_replays(bins):
    import torch
    from paper_2603_12016_amd import nyx
    rng = np.random.default_rng(bins)
    I = rng.integers(0, 60000, (1, 400, 420)).astype(np.uint16)
    y, x = np.mgrid[0:400, 0:420]
    L = ((y // 14) * 30 + x // 14 + 1).astype(np.uint32)[None]     # small regions
    for k in range(10):
        L[0, 300:360, 40 * k:40 * k + 40] = 5000 + k               # and ten of 2400 voxels
    images = [(torch.from_numpy(I.view(np.int16)).cuda(), torch.from_numpy(L.view(np.int32)).cuda())]
    torch.cuda.synchronize()
    ctx = nyx.nyx_create(0)
    offs = nyx.nyx_offsets_default(2, 1)
    plan = nyx.nyx_plan_create(ctx, images, bins, offs, nyx.NYX_FP64)
    print(nyx.nyx_plan_describe(plan), flush=True)
    a, b, c = (nyx.new_table(plan, len(offs), nyx.NYX_FP64) for _ in range(3))
    nyx.nyx_plan_execute(plan, a)
    nyx.nyx_plan_check(plan)
    want = a.cpu().numpy()

    def same(t):
        nyx.nyx_plan_check(plan)
        np.testing.assert_allclose(t.cpu().numpy(), want, rtol=1e-12, atol=1e-300)

    for _ in range(12):
        a.fill_(-7.0)
        nyx.nyx_plan_execute(plan, a)
        same(a)
    nyx.nyx_plan_execute_per_roi(plan, c)
    a.fill_(-7.0)
    nyx.nyx_plan_execute(plan, a)
    same(a)
    for k in range(9):
        for t in (a, b):
            t.fill_(-7.0)
        t = (a, b)[k & 1]
        nyx.nyx_plan_execute(plan, t)
        same(t)
        assert bool(((b, a)[k & 1] == -7.0).all())
    for k in range(6):          # a per-ROI pass between replays of the one branch
        a.fill_(-7.0)
        c.fill_(-7.0)
        nyx.nyx_plan_execute(plan, a)
        same(a)
        nyx.nyx_plan_execute_per_roi(plan, c)
        same(c)
    nyx.nyx_plan_profile(plan, c)
    for _ in range(6):
        a.fill_(-7.0)
        c.fill_(-7.0)
        nyx.nyx_plan_execute(plan, a)
        same(a)
        assert bool((c == -7.0).all())
