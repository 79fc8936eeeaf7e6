"""Edges of the gradient kernel behind the Hubbard forces and stress, against
the oracle: one and several points per thread, columns cut into chunks of
planes with a shorter last one, axes barely longer than the reach (every
plane wraps; the oracle takes no shorter ones), Bloch phases, lower orders.

Bars as for the other force and stress tests: 1e-10 (FP64) and 1e-4 (FP32
blocks) of the largest component.
"""
import numpy as np
import pytest

import workloads
from test_gpu_forces import _gpu, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,k", [("fp64", 0), ("mixed", 0), ("fp64", 1), ("mixed", 1)])
@pytest.mark.parametrize("n,n0", [((16, 12, 31), 6), ((13, 12, 25), 6), ((18, 10, 12), 5), ((12, 11, 7), 6),
                                  ((8, 20, 9), 3)])
def test_forces_and_stress_on_gradient_shapes(n, n0, precision, k):
    from oracle import forces as oforces
    cfg = workloads.make_config("tiny")
    cfg.update(n=np.array(n, np.int32), ns=5, n0=n0, nelec=4.0)
    if k:
        cfg["kpts"] = np.array([[0.11, 0.05, -0.13]])
    X, f = _inputs(cfg, 5)
    F, S, Xr = _gpu(cfg, precision, X, f)
    Fo, So = oforces.forces_and_stress(cfg, Xr, f)
    bar = 1e-10 if precision == "fp64" else 1e-4
    assert np.abs(F - Fo).max() < bar * np.abs(Fo).max()
    assert np.abs(S - So).max() < bar * np.abs(So).max()
