"""Edges of the projector pass against the CPU oracle: brick shapes (16 x 4,
8 x 8, blocks that end outside the row, runs of 64 points with a ragged last
brick, stacked planes or not), state counts around the 16 and 64 of a wave and
a workgroup, padded rows, and 3, 5 and 9 slot tiles per projection brick (the
last swept twice by the projection alone).

Bars of the operator and the filter as for the other operator tests: 1e-12 and
2e-6 of the largest value for H (summation order), 1e-11 and 3e-5 for a filter
of degree 3.
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


def _cell(n, ns, k, copies):
    cfg = workloads.make_config("tiny")
    rng = np.random.default_rng(5)
    pos = np.concatenate([np.asarray(cfg["pos"]) + (c > 0) * rng.normal(size=np.shape(cfg["pos"])) for c in range(copies)])
    cfg.update(n=np.array(n, np.int32), ns=ns, nelec=1.0, atom_species=np.tile(cfg["atom_species"], copies), pos=pos)
    if k:
        cfg["kpts"] = np.array([[0.11, 0.05, -0.13]])
    return cfg


@pytest.mark.parametrize("precision,k", [("fp64", 0), ("mixed", 0), ("fp64", 1), ("mixed", 1)])
@pytest.mark.parametrize("n,ns,pad,copies", [
    ((16, 16, 12), 17, 0, 1), ((20, 16, 9), 1, 3, 1), ((31, 12, 8), 15, 1, 1), ((11, 10, 9), 70, 5, 1),
    ((16, 8, 8), 33, 0, 2), ((23, 16, 9), 18, 0, 1), ((15, 8, 8), 16, 1, 4), ((13, 12, 10), 65, 0, 4)])
def test_projector_pass(n, ns, pad, copies, precision, k):
    torch = _torch()
    from oracle import chfsi
    from oracle.hamiltonian import Hamiltonian
    from paper_2507_23612_amd import hcu
    cfg = _cell(n, ns, k, copies)
    ctx = hcu.HcuContext(cfg, precision)
    rng = np.random.default_rng(3)
    D = rng.normal(size=(1, ctx.nhub, 5, 5)) * 0.05
    D = 0.2 * np.eye(5) + D + D.transpose(0, 1, 3, 2)
    ctx.set_hubbard_occupation(D)
    Xh = workloads.random_block(ctx.nd, ns, 3, bool(k))
    X = torch.full((ns, ctx.nd + pad), float("nan"), dtype=ctx.dtype, device="cuda")
    X[:, :ctx.nd] = torch.from_numpy(Xh).cuda().to(ctx.dtype)
    Xh = X[:, :ctx.nd].cpu().numpy().astype(np.complex128 if k else np.float64)
    H = Hamiltonian(cfg, cfg["kpts"][0] if k else (0.0, 0.0, 0.0), D=list(D[0]))
    want = H.apply(Xh)
    bounds = (4.0, 2.0 * float(np.abs(want).max()), -1.0)
    filtered = chfsi.cheb_filter(H.apply, Xh, 3, *bounds)
    Y = torch.empty_like(X)
    fp64 = precision == "fp64"
    for call, ref, tol in ((lambda: ctx.apply_h(X, Y), want, 1e-12 if fp64 else 2e-6),
                           (lambda: ctx.cheb_filter(X, Y, 3, *bounds), filtered, 1e-11 if fp64 else 3e-5)):
        Y.fill_(float("nan"))
        call()
        got = Y.cpu().numpy()
        assert np.isnan(got[:, ctx.nd:]).all()
        err = float(np.abs(got[:, :ctx.nd] - ref).max() / np.abs(ref).max())
        print(f"[gpu] projector pass {n} ns={ns} {precision} k={k}: {err:.1e}", flush=True)
        assert err < tol
    ctx.close()


def test_rounding_of_fp32_projections():
    """Forces and stress of FP32 blocks against FP64 ones of the same values, 12
    random blocks on each of three grids, real and complex: both are sums over
    projections, whose rounding they show.  Bars: the geometric means over the
    contexts of the rms errors that kernels with two (complex: four) chains of
    128 to 256 additions per projection brick left, 1.20e-6 and 1.29e-6."""
    torch = _torch()
    from paper_2507_23612_amd import hcu
    rms = []
    for n, k in (((36, 36, 24), 0), ((36, 36, 24), 1), ((31, 33, 20), 0), ((31, 33, 20), 1), ((32, 32, 20), 0),
                 ((32, 32, 20), 1)):
        cfg = workloads.make_config("c1")
        cfg["n"] = np.array(n, np.int32)
        if k:
            cfg["kpts"] = np.array([[0.11, 0.05, -0.13]])
        ctxs = [hcu.HcuContext(cfg, p) for p in ("mixed", "fp64")]
        for c in ctxs:
            c.set_hubbard_occupation(hcu.initial_occupation(c, cfg))
        occ = (1 / (1 + np.exp(np.linspace(-10, 10, cfg["ns"]))))[None, None, :]
        err = []
        for seed in range(12):
            X = torch.from_numpy(workloads.random_block(ctxs[0].nd, cfg["ns"], seed, bool(k))).cuda().to(ctxs[0].dtype)
            got = []
            for c in ctxs:
                c.set_start(0, 0, X.to(c.dtype), X[0].to(c.dtype).clone())
                got.append((c.hubbard_forces(occ), c.hubbard_stress(occ)))
            err.append([np.linalg.norm(a - b) / np.linalg.norm(b) for a, b in zip(*got)])
        rms.append(np.sqrt(np.mean(np.square(err), axis=0)))
        for c in ctxs:
            c.close()
    forces, stress = np.exp(np.mean(np.log(rms), axis=0))
    assert forces < 1.20e-6 and stress < 1.29e-6, (forces, stress)


def _chunks(H, points):
    """Chunks of 16 functions that touch each brick; points [brick][64]."""
    of = np.full(H.nd, -1)
    for b, p in enumerate(points):
        of[p] = b
    count = np.zeros(len(points), int)
    for a in H.atoms:
        for idx, vals in ((a["kb_idx"], a["kb_vals"]), (a["hub_idx"], a["hub_vals"]) if "hub_idx" in a else ((), ())):
            if len(idx):
                count[np.unique(of[idx])] += len(vals)
    return (count + 15) // 16


@pytest.mark.parametrize("layout,precision,k", [("runs", "fp64", 0), ("runs", "mixed", 0), ("runs", "fp64", 1),
                                                ("runs", "mixed", 1), ("stacks", "mixed", 0)])
def test_scatter_alone_past_an_empty_brick(layout, precision, k):
    """Enough states that the scatter alone takes whole groups of bricks, and in
    a group a brick of more than 16 functions, then one that no function
    touches, then one with functions again: its function list is the third
    brick's.  runs: 64 points each, four to a row, atoms apart in x; stacks:
    blocks of 16 x 4 points, two planes by five blocks in y, supports that meet
    the first plane of a pair last and one block of rows of it each."""
    torch = _torch()
    from oracle import chfsi
    from oracle.hamiltonian import Hamiltonian
    from paper_2507_23612_amd import hcu
    cfg = workloads.make_config("tiny")
    if layout == "runs":
        n, ns, h = (256, 17, 10), 420, 0.4
        pos = [(12.6, 2.0, 1.0), (13.1, 4.0, 2.0), (64.0, 3.0, 2.0)]
    else:
        n, ns, h = (32, 40, 32), 1000, 0.5
        pos = [(6.0 + 0.1 * i, 0.75, 3.7) for i in range(4)] + [(6.0, 2.75, 3.7)]
    cfg.update(n=np.array(n, np.int32), ns=ns, nelec=1.0, L=h * np.array(n), pos=np.array(pos),
               atom_species=np.zeros(len(pos), np.int32))
    if k:
        cfg["kpts"] = np.array([[0.02, 0.05, -0.13]])
    H = Hamiltonian(cfg, cfg["kpts"][0] if k else (0.0, 0.0, 0.0))
    grid = np.arange(H.nd).reshape(n[::-1])
    if layout == "runs":
        groups = grid.reshape(-1, 4, 64)
    else:   # [z pair][x block][y stack] groups of [y block][plane] bricks
        g = grid.reshape(16, 2, 2, 5, 4, 2, 16).transpose(0, 2, 5, 3, 1, 4, 6)
        groups = g.reshape(-1, 10, 64)
    c = _chunks(H, groups.reshape(-1, 64)).reshape(groups.shape[:2])
    met = [(a, b) for a in range(c.shape[0]) for b in range(c.shape[1] - 2)
           if c[a, b] >= 2 and c[a, b + 1] == 0 and c[a, b + 2:].any()]
    assert met
    ctx = hcu.HcuContext(cfg, precision)
    rng = np.random.default_rng(3)
    D = rng.normal(size=(1, ctx.nhub, 5, 5)) * 0.05
    D = 0.2 * np.eye(5) + D + D.transpose(0, 1, 3, 2)
    ctx.set_hubbard_occupation(D)
    H.set_occupation(list(D[0]))
    X = torch.from_numpy(workloads.random_block(ctx.nd, ns, 3, bool(k))).cuda().to(ctx.dtype)
    cols = [0, 63, 64, 200, ns - 1]
    Xh = X[cols].cpu().numpy().astype(np.complex128 if k else np.float64)
    want = H.apply(Xh)
    bounds = (4.0, 2.0 * float(np.abs(want).max()), -1.0)
    filtered = chfsi.cheb_filter(H.apply, Xh, 3, *bounds)
    Y = torch.empty_like(X)
    fp64 = precision == "fp64"
    for call, ref, tol in ((lambda: ctx.apply_h(X, Y), want, 1e-12 if fp64 else 2e-6),
                           (lambda: ctx.cheb_filter(X, Y, 3, *bounds), filtered, 1e-11 if fp64 else 3e-5)):
        Y.fill_(float("nan"))
        call()
        err = float(np.abs(Y[cols].cpu().numpy() - ref).max() / np.abs(ref).max())
        print(f"[gpu] scatter past an empty brick {layout} {precision} k={k}: {err:.1e}", flush=True)
        assert err < tol
    ctx.close()
