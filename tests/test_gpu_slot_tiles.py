"""GPU: the slot form for few right-hand sides (adaptive and float64 plans).

Up to 8 right-hand sides share tiles of 16 columns, (group, rhs) of neighbouring
groups; 9 or more take a slot per workgroup.  A column's translations are the
same bits in both; the leaf passes of another right-hand side count (the near
field on the MFMA from 4, other S2M and L2T forms) round differently: 1e-6
relative L2, as for batches."""
from __future__ import annotations

import os

import numpy as np
import pytest

from oracle.kernel import rel_l2
from paper_1311_4257_amd import workloads

pytestmark = pytest.mark.gpu

CACHE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), ".dfmm_cache")


def _dens(torch, n, nrhs, seed, cuda):
    g = torch.Generator(device=cuda).manual_seed(seed)
    return torch.view_as_complex(torch.randn((nrhs, n, 2), generator=g, device=cuda, dtype=torch.float64))


def test_more_tiles_than_grid_y_takes(cuda):
    """133,000 boxes and more on one level make over 65,536 tiles at 8 right-hand
    sides, more than grid y takes.  The points fill a disc, one per box of width
    1/128, so that a box has about 27 M2L pairs."""
    import torch

    from paper_1311_4257_amd import dfmm

    i, j = [v.ravel() for v in np.meshgrid(np.arange(512), np.arange(512))]
    disc = (i - 255.5) ** 2 + (j - 255.5) ** 2 < 206.0 ** 2
    box = np.stack([i, j, np.full_like(i, 256)], axis=1)[disc]
    pts = (box + 0.25 + 0.5 * np.random.default_rng(31).random(box.shape)) / 128.0 - 2.0
    assert len(pts) > 2 * 65536 + 8
    plan = dfmm.Plan(pts, 4.0, eps=1e-2, cache_dir=CACHE, device=0, leaf_max=1, lf_levels=6)
    info = plan.info()
    assert info.leaves == len(pts) and info.depth_max - info.depth == 6
    f = _dens(torch, len(pts), 9, 32, cuda).to(torch.complex64)
    wide = plan.apply(f).cpu().numpy()
    u = torch.empty((8, len(pts)), dtype=torch.complex64, device=cuda)
    for _ in range(2):
        u.zero_()
        plan.apply(f[:8].contiguous(), u)
        got = u.cpu().numpy()
        for k in range(8):
            assert rel_l2(got[k], wide[k]) < 1e-6
