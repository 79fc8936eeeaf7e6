"""The Lanczos bound's device-side recursion against the oracle: one step, as
many as one batch of scalars holds and one more, all block types, and the
start vectors that it refuses.

FP64 bar 1e-9 of the bound (a recursion of 25 steps on vectors of 1e3 points);
FP32 1e-4 (each step's vectors rounded at 6e-8, amplified by the recursion).
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("precision,k", [("fp64", 0), ("mixed", 0), ("fp64", 1), ("mixed", 1)])
def test_lanczos_steps(precision, k):
    torch = _torch()
    from oracle import chfsi
    from oracle.hamiltonian import Hamiltonian
    from paper_2507_23612_amd import hcu
    cfg = workloads.make_config("tiny")
    if k:
        cfg["kpts"] = np.array([[0.11, 0.05, -0.13]])
    ctx = hcu.HcuContext(cfg, precision)
    D = hcu.initial_occupation(ctx, cfg)
    ctx.set_hubbard_occupation(D)
    H = Hamiltonian(cfg, cfg["kpts"][0] if k else (0.0, 0.0, 0.0), D=list(D[0]))
    X = torch.from_numpy(workloads.random_block(ctx.nd, ctx.ns, 3, bool(k))).cuda().to(ctx.dtype)
    v0 = X[0].clone()
    ctx.set_start(0, 0, X, v0)
    vh = v0.cpu().numpy().astype(np.complex128 if k else np.float64)
    bar = 1e-9 if precision == "fp64" else 1e-4
    for steps in (1, 2, 10, 24, 25):
        tmin, b = ctx.lanczos_bounds(0, 0, steps)
        wmin, wb = chfsi.lanczos(H.apply, vh, steps)
        assert abs(tmin - wmin) < bar * wb and abs(b - wb) < bar * wb, steps
    for bad in (0.0, float("nan")):
        ctx.set_start(0, 0, X, torch.full_like(v0, bad))
        with pytest.raises(hcu.HcuError):
            ctx.lanczos_bounds(0, 0, 10)
    ctx.close()


@pytest.mark.parametrize("n,k", [((36, 36, 24), 0), ((31, 33, 20), 0), ((40, 28, 22), 0), ((36, 36, 24), 1)])
def test_lowest_ritz_value_of_fp32_blocks(n, k):
    """The lowest Ritz value of FP32 blocks against the FP64 oracle, 20 start
    vectors: the vectors are doubles, so only the projector term rounds in 32
    bits.  Its norm is at most the largest coupling, 1 Ha; the table, the
    projections, the coupled projections and the result round it by at most
    4e-7 of that together, which bounds the shift of a Ritz value in Ha."""
    torch = _torch()
    from oracle import chfsi
    from oracle.hamiltonian import Hamiltonian
    from paper_2507_23612_amd import hcu
    cfg = workloads.make_config("c1")
    cfg["n"] = np.array(n, np.int32)
    if k:
        cfg["kpts"] = np.array([[0.11, 0.05, -0.13]])
    ctx = hcu.HcuContext(cfg, "mixed")
    D = hcu.initial_occupation(ctx, cfg)
    ctx.set_hubbard_occupation(D)
    H = Hamiltonian(cfg, cfg["kpts"][0], D=list(D[0]))
    X = torch.from_numpy(workloads.random_block(ctx.nd, max(20, ctx.ns), 11, bool(k))).cuda().to(ctx.dtype)
    for i in range(20):
        ctx.set_start(0, 0, X[:ctx.ns], X[i].clone())
        got, b = ctx.lanczos_bounds(0, 0, 10)
        want, wb = chfsi.lanczos(H.apply, X[i].cpu().numpy().astype(np.complex128 if k else np.float64), 10)
        assert abs(got - want) < 4e-7 and abs(b - wb) < 4e-7, (i, got - want, b - wb)
    ctx.close()
