"""The symmetric run where the Gram products' rows are split over thousands of partial sums
of few elements, over some, and over too few to share a sum between threads: against the
oracle's vector-by-vector form."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# (sites, vectors, steps): 2048, 2048, 1024, 683, 64 and 32 splits; one element, a part of a
# 16-element block, one block of steps, and a block with a remainder
@pytest.mark.parametrize("n,R,steps", [(17, 2, 1), (17, 2, 5), (16, 4, 32), (17, 2, 33), (12, 2, 20), (11, 4, 33)])
@pytest.mark.parametrize("precision", [0, 1])
def test_splits_match_oracle(n, R, steps, precision):
    import paper_2607_25585_amd as F
    rng = np.random.default_rng(n)
    sysm = W.System(two_s=np.ones(n, np.int32), J=W.ring_couplings(n, 1.0), d=None, e=np.tile([0.0, 0.0, 1.0], (n, 1)),
                    g=rng.uniform(1.5, 2.5, n), B=np.array([0.3, 0.2, 1.0]), pos=None)
    T = np.array([1.0, 5.0, 40.0])
    print("case splits", n, R, steps, precision, flush=True)
    got = F.run_sftlm(F.Hamiltonian(sysm), R, steps, T, seed=4, precision=precision)
    want = of.sftlm(sysm, R, steps, T, seed=4)[0]
    for k in ("lnZ", "E", "C", "M"):
        floor = 1e-3 * np.max(np.abs(want[k])) + 1e-300
        err = np.max(np.abs(got[k][0] - want[k]) / np.maximum(np.abs(want[k]), floor))
        assert err < (1e-3 if precision else 1e-8), k
