"""GPU: densities far below 1 keep the accuracy of their plan.

The translation GEMMs hold a float32 in three bfloat16 parts, whose last part needs
2^-102; a right-hand side without a density from 2^-63 up is scaled by 2^64 through
them.  A pass is linear, so densities scaled by a power of two must give the
potentials scaled by it, up to what float32 loses near its own lower end:

* 2^-105: densities and products are normal numbers; sums that cancel round at
  2^-150, 2^-45 of the densities: 1e-9 relative L2 is 3 x 10^4 of those.
* 2^-118: products round at 2^-150, 2^-32 of the densities, over the some hundred
  products of a leaf's passes: 1e-7, within 2e-7 (an eps = 1e-6 plan, whose bound
  is 1e-6)."""
from __future__ import annotations

import os

import pytest

from paper_1311_4257_amd import workloads

pytestmark = pytest.mark.gpu

CACHE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), ".dfmm_cache")


def _dens(torch, n, nrhs, seed, cuda):
    g = torch.Generator(device=cuda).manual_seed(seed)
    return torch.view_as_complex(torch.randn((nrhs, n, 2), generator=g, device=cuda))


def _scaled(torch, f, e):
    return torch.view_as_complex((torch.view_as_real(f).double() * 2.0**e).float())


def _err(torch, u, e, ref):
    u, ref = u.to(torch.complex128) * 2.0**-e, ref.to(torch.complex128)
    return (torch.linalg.norm(u - ref) / torch.linalg.norm(ref)).item()


def _plan(kind):
    from paper_1311_4257_amd import dfmm

    if kind == "adaptive":
        return dfmm.Plan(workloads.sphere_points(8000, 4.0, 61), 4.0, eps=1e-4, cache_dir=CACHE, device=0, leaf_max=32)
    eps = 1e-6 if kind == "precise" else 1e-4
    return dfmm.Plan(workloads.sphere_points(3000, 4.0, 62), 4.0, eps=eps, cache_dir=CACHE, device=0)


# few right-hand sides, the batched leaf passes, the tiled permutations, the slot form
@pytest.mark.parametrize("nrhs", [1, 4, 17, 32])
@pytest.mark.parametrize("kind", ["fast", "precise", "adaptive"])
def test_scaled_densities_give_scaled_potentials(cuda, kind, nrhs):
    import torch

    plan = _plan(kind)
    f = _dens(torch, plan.N, nrhs, 63, cuda)
    ref = plan.apply(f)
    for e, bound in ((-60, 1e-9), (-66, 1e-9), (-105, 1e-9), (-118, 2e-7)):
        assert _err(torch, plan.apply(_scaled(torch, f, e)), e, ref) < bound, e
    assert torch.equal(plan.apply(f), ref)


def test_the_scale_is_of_one_apply_and_one_right_hand_side(cuda):
    """Right-hand sides of very different sizes in one apply, and applies of different
    sizes after each other in one workspace of any contents, eager and as a graph."""
    import torch

    plan = _plan("fast")
    f = _dens(torch, plan.N, 3, 64, cuda)
    mixed = f.clone()
    mixed[1] = _scaled(torch, f[1], -105)
    small = _scaled(torch, f, -105)
    ref = plan.apply(f)
    ws = torch.full((plan.workspace_bytes(3),), 0x15, dtype=torch.uint8, device=cuda)
    x, u = torch.empty_like(f), torch.empty_like(f)

    def check(run):
        for y, e in ((small, (-105,) * 3), (f, (0, 0, 0)), (mixed, (0, -105, 0)), (small, (-105,) * 3)):
            x.copy_(y)
            torch.cuda.synchronize()
            run()
            torch.cuda.synchronize()
            for k in range(3):
                assert _err(torch, u[k], e[k], ref[k]) < 1e-9, (e, k)

    check(lambda: plan.apply_ws(x, u, ws))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.apply_ws(x, u, ws)
    check(graph.replay)


def test_not_finite_densities_stay_in_their_right_hand_side(cuda):
    import torch

    plan = _plan("fast")
    f = _dens(torch, plan.N, 3, 65, cuda)
    ref = plan.apply(f)
    for bad in (float("inf"), float("nan")):
        g = f.clone()
        g[1, 7] = bad
        u = plan.apply(g)
        assert torch.equal(u[0], ref[0]) and torch.equal(u[2], ref[2])
        assert not torch.isfinite(torch.view_as_real(u[1])).any()
