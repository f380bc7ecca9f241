"""The symmetric run's waves of interleaved vectors and its Gram products on the
matrix cores, at the edges: one pair, an odd number of pairs, a last wave that is
smaller than the others, steps around the 32-wide blocks, few and many rows per
split, complex64, against the oracle's vector-by-vector form."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _check(sysm, R, steps, seed, fields=None, precision=0, tol=1e-8):
    import paper_2607_25585_amd as F
    T = np.array([0.3, 1.0, 5.0, 40.0])
    print("case", sysm.two_s.tolist(), R, steps, precision, flush=True)
    got = F.run_sftlm(F.Hamiltonian(sysm), R, steps, T, seed=seed, fields=fields, precision=precision)
    ref = of.sftlm(sysm, R, steps, T, seed=seed, fields=fields)
    for f, want in enumerate(ref):
        for k in ("lnZ", "E", "C", "M"):
            floor = 1e-3 * np.max(np.abs(want[k])) + 1e-300
            assert np.max(np.abs(got[k][f] - want[k]) / np.maximum(np.abs(want[k]), floor)) < tol, k


@pytest.mark.parametrize("R,steps", [(2, 1), (2, 31), (4, 32), (6, 33), (14, 64), (20, 65)])
@pytest.mark.parametrize("n,two_s", [(3, 3), (4, 5)])
def test_waves_match_oracle(n, two_s, R, steps):
    rng = np.random.default_rng(n)
    sysm = W.random_small_system(rng, n, max_two_s=two_s)
    sysm.two_s[:] = two_s
    _check(sysm, R, min(steps, (two_s + 1) ** n // 2), 5)


def test_last_wave_smaller_and_second_field():
    # 4^8 rows, 60 steps: eight vectors' bases fit the limit, so 8 + 2 vectors
    sysm = W.cfg5_system(W.cfg5_params(3)[1])
    _check(sysm, 10, 60, 7)
    small = W.ring_sftlm(4, 0.7)[0]
    _check(small, 6, 40, 7, fields=[[0.1, 0.2, 0.3], [0.0, 1.0, 0.0]])


def test_single_precision_storage():
    _check(W.ring_sftlm(4, 1.0)[0], 6, 40, 9, precision=1, tol=1e-3)
