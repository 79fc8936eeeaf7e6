"""The Rayleigh-Ritz eigensolve of small blocks (one workgroup, in LDS): odd
and even sizes around its limits of 32 and 64 states and one past them,
against scipy's generalized eigensolver, and a degenerate Gram matrix.

Bars as for the larger sizes: Ritz values 1e-10 of the spectral width, the
rotated block orthonormal and diagonalising H to 1e-10.
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


def _context(ns, k):
    from paper_2507_23612_amd import hcu
    cfg = workloads.make_config("tiny")
    cfg.update(ns=ns, nelec=1.0, first_passes=1)
    if k:
        cfg["kpts"] = np.array([[0.18, -0.18, 0.28]])
    ctx = hcu.HcuContext(cfg)
    ctx.set_hubbard_occupation(hcu.initial_occupation(ctx, cfg))
    return cfg, ctx


@pytest.mark.parametrize("k", [0, 1])
@pytest.mark.parametrize("ns", [1, 2, 3, 17, 31, 32, 33, 63, 64, 65])
def test_small_eigensolve_matches_scipy(ns, k):
    torch = _torch()
    import scipy.linalg
    cfg, ctx = _context(ns, k)
    X0 = torch.from_numpy(workloads.random_block(ctx.nd, ns, 3, bool(k))).cuda().to(ctx.dtype)
    ctx.set_start(0, 0, X0, X0[0].clone())
    tmin, b = ctx.lanczos_bounds(0, 0, 10)
    a = tmin + (b - tmin) / 10.0
    Y = torch.empty_like(X0)
    ctx.cheb_filter(X0, Y, m=int(cfg["degree"]), a=a, b=b, aL=tmin)
    HY = torch.empty_like(Y)
    ctx.apply_h(Y, HY)
    S, Hs = ctx.gram(Y, HY)
    want = scipy.linalg.eigh(Hs, S, eigvals_only=True)
    ctx.chfsi_pass(0, 0)
    X = ctx.get_orbitals(0, 0)
    HX = torch.empty_like(X)
    ctx.apply_h(X, HX)
    Sx, Hx = ctx.gram(X, HX)
    ctx.close()
    lam = np.real(np.diag(Hx))
    width = max(want[-1] - want[0], 1.0)
    assert np.max(np.abs(lam - want)) < 1e-10 * width
    assert np.max(np.abs(Sx - np.eye(ns))) < 1e-10
    assert np.max(np.abs(Hx - np.diag(lam))) < 1e-10 * width


@pytest.mark.parametrize("k", [0, 1])
def test_dependent_states_are_refused(k):
    torch = _torch()
    from paper_2507_23612_amd import hcu
    _, ctx = _context(20, k)
    X0 = torch.from_numpy(workloads.random_block(ctx.nd, 20, 3, bool(k))).cuda().to(ctx.dtype)
    X0[7] = 0.0
    ctx.set_start(0, 0, X0, X0[0].clone())
    ctx.lanczos_bounds(0, 0, 10)
    with pytest.raises(hcu.HcuError):
        ctx.chfsi_pass(0, 0)
    ctx.close()
