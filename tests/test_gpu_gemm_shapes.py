"""GPU: shapes of the translation GEMMs that a plan of ordinary skeletons seldom takes.

Bounds as in test_gpu_gemm_edges: a pass over given skeletons stays within tens of
float32 roundings of its float64 value, 1e-6 relative L2; where only the launch
differs, the bits are the same."""
from __future__ import annotations

import glob

import numpy as np
import pytest

from oracle import fmm as F
from oracle import operators as O
from oracle.kernel import rel_l2
from oracle.tree import build_structure
from paper_1311_4257_amd import workloads
from tests.helpers import inject, oracle_opset

pytestmark = pytest.mark.gpu


def _dens(torch, n, nrhs, seed, cuda):
    g = torch.Generator(device=cuda).manual_seed(seed)
    return torch.view_as_complex(torch.randn((nrhs, n, 2), generator=g, device=cuda, dtype=torch.float64))


def _truncated(tau, rank_hf, rank_lf):
    """The oracle's tau = 1e-3 skeletons cut to the given ranks, in a set of another tau."""
    from paper_1311_4257_amd import dfmm

    ops = oracle_opset(1e-3, 2)
    s = dfmm.OpSet.create(tau, ops.w_hi)

    def put(w, d, sk, r):
        r = min(r, len(sk.a))
        s.set(w, d, sk.a[:r], sk.b[:r], sk.D[:r, :r] / np.linalg.norm(sk.D[:r, :r]))

    for w, sks in ops.hf.items():
        for d, sk in enumerate(sks):
            put(float(w), d, sk, rank_hf)
    put(0.5, 0, ops.lf, rank_lf)
    return s


@pytest.mark.parametrize("rank", [5, 8, 11, 17, 24, 27, 33, 40])
@pytest.mark.parametrize("nrhs", [1, 3, 17])
def test_precise_plans_at_tile_edges(cuda, rank, nrhs):
    """Precise plans (tau < 3e-6): the directional operators in four planes."""
    import torch

    from paper_1311_4257_amd import dfmm

    ops = _truncated(1e-6, rank, rank + 3)
    pts = workloads.sphere_points(1500, 8.0, 91)
    f = _dens(torch, len(pts), nrhs, 92, cuda)
    exact = dfmm.Plan(pts, 8.0, opset=ops, device=0, precision=dfmm.PREC_FP64).apply(f).cpu().numpy()
    u = dfmm.Plan(pts, 8.0, opset=ops, device=0).apply(f.to(torch.complex64)).cpu().numpy().astype(np.complex128)
    assert rel_l2(u, exact) < 1e-6


@pytest.mark.parametrize("nrhs,prec,tau", [(1, 0, 1e-3), (5, 0, 1e-3), (1, 1, 1e-3), (5, 2, 1e-3), (3, 0, 1e-6)])
def test_six_to_eight_waves_do_not_change_results(cuda, tmp_path, nrhs, prec, tau):
    """Workgroups of 6 to 8 waves, forced through the tuning record (tile width,
    slices, an unused number, waves)."""
    import torch

    from paper_1311_4257_amd import dfmm

    pts, _, cfg = workloads.make_config("sphere4", N=2048)
    ops = inject(oracle_opset(tau, 1))
    f = _dens(torch, len(pts), nrhs, 707, cuda).to(torch.complex64)
    ref = dfmm.Plan(pts, cfg["K"], opset=ops, cache_dir=str(tmp_path), device=0, precision=prec).apply(f)
    (rec,) = glob.glob(str(tmp_path / "dfmm_tune_*.txt"))
    n = int(open(rec).read().split()[2])
    for nw in (6, 7, 8):
        for nt, sl in ((1, 1), (2, 2), (3, 1), (4, 1)):
            text = f"dfmm-tune 4 {n}\n" + f"{nt} {sl} 0 {nw}\n" * n + "fused 0\n"
            with open(rec, "w") as fh:
                fh.write(text)
            plan = dfmm.Plan(pts, cfg["K"], opset=ops, cache_dir=str(tmp_path), device=0, precision=prec)
            assert torch.equal(plan.apply(f), ref), (nt, sl, nw)
            assert open(rec).read() == text, "the forced shape was not taken"


def test_one_or_two_reductions_of_a_level(cuda):
    """The L2L and M2L pairs of a level are reduced in one pass up to 64 MB of L2L
    outputs.  The K = 16 sphere crosses that between 5 and 15 right-hand sides, whose
    other passes are the same: a column's bits do not depend on it."""
    import torch

    from paper_1311_4257_amd import dfmm

    pts = workloads.sphere_points(16384, 16.0, 94)
    plan = dfmm.Plan(pts, 16.0, opset=inject(oracle_opset(1e-3, 4)), device=0)
    f = _dens(torch, len(pts), 15, 95, cuda).to(torch.complex64)
    assert torch.equal(plan.apply(f[:5].contiguous()), plan.apply(f)[:5])


@pytest.mark.parametrize("tau", [1e-3, 1e-6])
@pytest.mark.parametrize("rank", [829, 837])
def test_ranks_whose_columns_do_not_fit(cuda, rank, tau):
    """Up to rank 832 16 columns of three planes fit LDS, past it a chunk has 8.  Two
    clusters that see each other through one pair of boxes at width 1; the far field of
    one in the other against the oracle's pass over the same skeletons."""
    import torch

    from paper_1311_4257_amd import dfmm

    rng = np.random.default_rng(rank)
    box = 0.05 * rng.random((40, 3)) + 0.1
    pts = np.concatenate([box - [1.7, 0, 0], box + [1.5, 0, 0]])
    st = build_structure(pts, 4.0)
    assert st.w_top == 1 and len(st.lists[st.tree.D - 1].tgt) == 2

    def skeleton(r, w):
        a = rng.standard_normal((r, 3))
        a *= (2.0 * w + rng.random((r, 1))) / np.linalg.norm(a, axis=1, keepdims=True)
        D = rng.standard_normal((r, r)) + 1j * rng.standard_normal((r, r))
        return O.Skeleton(a, (rng.random((r, 3)) - 0.5) * w, D / np.linalg.norm(D))

    ops = O.OpSet(tau, 1, {1: [skeleton(rank, 1.0) for _ in range(6)]}, skeleton(40, 0.5))
    plan = dfmm.Plan(pts, 4.0, opset=inject(ops), device=0)
    for nrhs in (1, 3, 20, 32):
        f = rng.standard_normal((nrhs, 80)) + 1j * rng.standard_normal((nrhs, 80))
        f[:, 40:] = 0.0
        f = f.astype(np.complex64)
        u = plan.apply(torch.from_numpy(f).to(cuda)).cpu().numpy()
        ref = F.fmm_apply(st, ops, f.astype(np.complex128))
        assert rel_l2(u[:, 40:], ref[:, 40:]) < 1e-6, nrhs
