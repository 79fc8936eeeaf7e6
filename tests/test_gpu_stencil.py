"""Edges of the stencil kernel against the CPU oracle: points per thread side
by side in x (vectors of two and four) or stacked in y, x halo from the tile
row or from memory, ragged tiles in x and y, z chunks of one plane and
shorter than the stencil's reach, grids narrower than the reach, and the
built-in shape on each.

FP64 bar 1e-12 of the largest value (summation order); FP32 2e-6 (about 40
terms of weights summing to 2.5 times the result's scale, rounded at 6e-8).
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


def _bare(n, ns, n0, k):
    """A cell without atoms: H is the kinetic stencil."""
    cfg = workloads.make_config("tiny")
    cfg.update(n=np.array(n, np.int32), ns=ns, n0=n0, nelec=1.0, L=0.3 * np.array(n, float),
               atom_species=np.zeros(0, np.int32), pos=np.zeros((0, 3)))
    if k:
        cfg["kpts"] = np.array([[0.11, 0.05, -0.13]])
    return cfg


@pytest.mark.parametrize("n,precision,k,n0", [
    ((20, 18, 14), "fp64", 0, 6), ((22, 16, 11), "mixed", 0, 6), ((64, 30, 7), "mixed", 0, 6),
    ((21, 17, 9), "fp64", 0, 6), ((20, 18, 14), "fp64", 1, 6), ((22, 16, 11), "mixed", 1, 6),
    ((13, 11, 10), "mixed", 1, 4), ((7, 6, 5), "fp64", 0, 6), ((23, 21, 9), "mixed", 0, 6), ((19, 16, 8), "fp64", 0, 4),
    ((20, 18, 14), "mixed", 0, 4), ((20, 18, 14), "fp64", 0, 5), ((16, 14, 9), "mixed", 0, 3), ((18, 14, 9), "mixed", 1, 1)])
def test_stencil_shapes(n, precision, k, n0):
    torch = _torch()
    from oracle import chfsi
    from oracle.hamiltonian import Hamiltonian
    from paper_2507_23612_amd import hcu
    cfg = _bare(n, 5, n0, k)
    ctx = hcu.HcuContext(cfg, precision)
    X = torch.from_numpy(workloads.random_block(ctx.nd, 5, 3, bool(k))).cuda().to(ctx.dtype)
    Xh = X.cpu().numpy().astype(np.complex128 if k else np.float64)
    H = Hamiltonian(cfg, cfg["kpts"][0])
    want = H.apply(Xh)
    bounds = (4.0, 2.0 * float(np.abs(want).max()), -1.0)
    filtered = chfsi.cheb_filter(H.apply, Xh, 3, *bounds)
    tol = 1e-12 if precision == "fp64" else 2e-6
    Y = torch.empty_like(X)
    shapes = [None] + [(tx, tyt, ry, tz) for ry in (1, 2, 4) for tx in (n[0], 8, 16, 36) for tyt in (1, 3, 4)
                       for tz in (n[2], 1, 5)]
    done = 0
    for sh in shapes:
        if sh is None:
            ctx.set_tuning(0)
        else:
            try:
                ctx.set_tuning(*sh)
            except hcu.HcuError:
                continue   # not admitted on this grid
        done += 1
        for got, ref in ((lambda: ctx.apply_h(X, Y), want), (lambda: ctx.cheb_filter(X, Y, 3, *bounds), filtered)):
            Y.fill_(float("nan"))
            got()
            err = float(np.abs(Y.cpu().numpy() - ref).max() / np.abs(ref).max())
            assert err < tol, (sh, err)
    assert done > 5
    ctx.close()


@pytest.mark.parametrize("precision,k", [("fp64", 0), ("mixed", 0), ("mixed", 1)])
def test_stencil_points_per_thread_agree_on_a_full_chip(precision, k):
    """Enough states to fill the device: two and four points per thread sum in
    the same order, so they agree to the last bit, and single complex points
    too (single real points are summed in another order: 1e-13 / 1e-5)."""
    torch = _torch()
    from paper_2507_23612_amd import hcu
    cfg = _bare((72, 72, 24), 192, 6, k)
    ctx = hcu.HcuContext(cfg, precision)
    g = torch.Generator(device="cuda").manual_seed(4)
    X = torch.randn((192, ctx.nd), generator=g, device="cuda", dtype=torch.float64).to(ctx.dtype)
    Y, ref = torch.empty_like(X), None
    for shape in ((72, 3, 2, 24), (72, 3, 4, 24), (36, 6, 4, 24), (32, 8, 4, 12), (72, 3, 1, 24), (36, 6, 1, 7)):
        ctx.set_tuning(*shape)
        for _ in range(2):
            Y.fill_(float("nan"))
            ctx.cheb_filter(X, Y, 3, 20.0, 190.0, -1.0)
            if ref is None:
                ref = Y.clone()
            if shape[2] == 1 and not k:
                assert float((Y - ref).abs().max() / ref.abs().max()) < (1e-13 if precision == "fp64" else 1e-5), shape
            else:
                assert torch.equal(Y, ref), shape
    ctx.close()


@pytest.mark.parametrize("n", [(36, 36, 24), (35, 33, 26)])
@pytest.mark.parametrize("k,n0", [(0, 6), (1, 6), (0, 4), (1, 4)])
def test_stencil_fp32_error(n, k, n0):
    """Rounding of one FP32 application to random blocks.  On random values the
    centre term makes most of the result, so only the centre and the n0 planes
    added after it round at the result's size; the neighbour sums (0.43 of it,
    most of that from the last two terms) and the rounded weights count as five
    more.  A rounding is 2.5e-8 rms of the value it is made at."""
    torch = _torch()
    from oracle.hamiltonian import Hamiltonian
    from paper_2507_23612_amd import hcu
    cfg = _bare(n, 8, n0, k)
    ctx = hcu.HcuContext(cfg, "mixed")
    X = torch.from_numpy(workloads.random_block(ctx.nd, 8, 7, bool(k))).cuda().to(ctx.dtype)
    Y = torch.empty_like(X)
    ctx.apply_h(X, Y)
    want = Hamiltonian(cfg, cfg["kpts"][0]).apply(X.cpu().numpy().astype(np.complex128 if k else np.float64))
    err = np.linalg.norm(Y.cpu().numpy() - want) / np.linalg.norm(want)
    ctx.close()
    assert err < 2.5e-8 * np.sqrt(n0 + 6), err


@pytest.mark.parametrize("shape", [(48, 4, 4), (36, 5, 4), (24, 6, 4), (32, 5, 4), (20, 8, 4), (16, 12, 4), (16, 16, 4)])
def test_stencil_halo_of_partial_rows(shape):
    """FP32, order 12: tiles that do not span the row, whose halo takes more
    vectors than threads although it has at most four values for each."""
    torch = _torch()
    from oracle.hamiltonian import Hamiltonian
    from paper_2507_23612_amd import hcu
    cfg = _bare((52, 64, 9), 3, 6, 0)
    ctx = hcu.HcuContext(cfg, "mixed")
    X = torch.from_numpy(workloads.random_block(ctx.nd, 3, 5, False)).cuda().to(ctx.dtype)
    Y = torch.empty_like(X)
    want = Hamiltonian(cfg, cfg["kpts"][0]).apply(X.cpu().numpy().astype(np.float64))
    for tz in (9, 4):
        ctx.set_tuning(*shape, tz)
        Y.fill_(float("nan"))
        ctx.apply_h(X, Y)
        assert float(np.abs(Y.cpu().numpy() - want).max() / np.abs(want).max()) < 2e-6
    ctx.close()
