"""GPU: the slot form for few right-hand sides (adaptive and float64 plans).

Up to 8 right-hand sides share tiles of 16 columns, (group, rhs) of neighbouring
groups; 9 or more take a slot per workgroup.  A column's translations are the
same bits in both.  In float64 so is the whole pass; in float32 the leaf passes of
another right-hand side count (the near field on the MFMA from 4, other S2M and
L2T forms) round differently: 1e-6 relative L2, as for batches."""
from __future__ import annotations

import os

import numpy as np
import pytest

from oracle.kernel import rel_l2
from paper_1311_4257_amd import workloads
from tests.helpers import inject, oracle_opset

pytestmark = pytest.mark.gpu

CACHE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), ".dfmm_cache")


def _dens(torch, n, nrhs, seed, cuda, dtype=None):
    g = torch.Generator(device=cuda).manual_seed(seed)
    f = torch.view_as_complex(torch.randn((nrhs, n, 2), generator=g, device=cuda, dtype=torch.float64))
    return f.to(dtype) if dtype else f


@pytest.fixture(scope="module")
def disc():
    """133,344 points on a disc, one per box of width 1/128 (27 M2L pairs each): over
    65,536 tiles at 8 right-hand sides, more than grid y takes, and levels long
    enough for tiles of 16 groups at one."""
    from paper_1311_4257_amd import dfmm

    i, j = [v.ravel() for v in np.meshgrid(np.arange(512), np.arange(512))]
    inside = (i - 255.5) ** 2 + (j - 255.5) ** 2 < 206.0 ** 2
    box = np.stack([i, j, np.full_like(i, 256)], axis=1)[inside]
    pts = (box + 0.25 + 0.5 * np.random.default_rng(31).random(box.shape)) / 128.0 - 2.0
    plan = dfmm.Plan(pts, 4.0, eps=1e-2, cache_dir=CACHE, device=0, leaf_max=1, lf_levels=6)
    info = plan.info()
    assert info.leaves == len(pts) and info.depth_max - info.depth == 6
    assert info.boxes[info.depth_max] > 2 * 65536
    return plan, len(pts)


@pytest.mark.parametrize("nrhs", [8, 5, 3, 2, 1])
def test_adaptive_tiles_of_many_groups(cuda, disc, nrhs):
    import torch

    plan, n = disc
    f = _dens(torch, n, 9, 32, cuda, torch.complex64)
    wide = plan.apply(f).cpu().numpy()
    u = plan.apply(f[:nrhs].contiguous()).cpu().numpy()
    for k in range(nrhs):
        assert rel_l2(u[k], wide[k]) < 1e-6


@pytest.mark.parametrize("nrhs", range(1, 9))
def test_float64_tiles_give_the_general_form(cuda, nrhs):
    import torch

    from paper_1311_4257_amd import dfmm

    pts = workloads.sphere_points(6000, 8.0, 98)
    plan = dfmm.Plan(pts, 8.0, opset=inject(oracle_opset(1e-3, 2)), device=0, precision=dfmm.PREC_FP64)
    f = _dens(torch, len(pts), 9, 99, cuda)
    assert torch.equal(plan.apply(f[:nrhs].contiguous()), plan.apply(f)[:nrhs])


@pytest.mark.parametrize("kind", ["adaptive", "fp64"])
def test_first_apply_takes_no_device_memory(cuda, kind):
    """In the caller's workspace the first apply of each number of right-hand sides
    allocates nothing: not even while another stream is being captured, where an
    allocation is refused."""
    import torch

    from paper_1311_4257_amd import dfmm

    pts = workloads.sphere_points(20000, 4.0, 101)

    def make():
        if kind == "fp64":
            return dfmm.Plan(pts, 4.0, opset=inject(oracle_opset(1e-3, 1)), device=0, precision=dfmm.PREC_FP64)
        return dfmm.Plan(pts, 4.0, eps=1e-4, cache_dir=CACHE, device=0, leaf_max=24)

    dt = torch.complex128 if kind == "fp64" else torch.complex64
    f = _dens(torch, len(pts), 8, 102, cuda, dt)
    old, new = make(), make()
    ws = torch.empty(new.workspace_bytes(8), dtype=torch.uint8, device=cuda)
    ref = {n: torch.empty_like(f[:n]) for n in range(1, 9)}
    got = {n: torch.empty_like(f[:n]) for n in range(1, 9)}
    for n in range(1, 9):
        old.apply_ws(f[:n].contiguous(), ref[n], ws)
    parts = {n: f[:n].contiguous() for n in range(1, 9)}
    x = torch.ones(16, device=cuda)
    side = torch.cuda.Stream(device=cuda)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for n in range(1, 8):
        new.apply_ws(parts[n], got[n], ws)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x += 1.0
        new.apply_ws(parts[8], got[8], ws, stream=side)  # side is not being captured
    torch.cuda.synchronize()
    for n in range(1, 9):
        assert torch.equal(got[n], ref[n])
