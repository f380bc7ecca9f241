"""The general-radix direct gather at the edges of its mapping: rows that do not fill
a tile, every number of lanes per row that the size rule gives, column counts that
group unevenly, sites past the sixteenth (second digit word), few and many pair
terms, with and without s+- s^z pieces; complex128 and complex64, elementwise
against the oracle, and a run through the Lanczos epilogue's column sums."""
import numpy as np
import pytest

import ftlm_workloads as W
from oracle import ftlm as of

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _mixed(two_s, seed, dipolar):
    rng = np.random.default_rng(seed)
    sysm = W.random_small_system(rng, len(two_s), dipolar=dipolar)
    sysm.two_s[:] = two_s
    if not dipolar:
        sysm.J[rng.random(sysm.J.shape) < 0.5] = 0.0
    return sysm


SYSTEMS = [
    ([1], 0), ([1, 2], 1), ([15, 15], 1), ([2] * 6, 1), ([1, 3, 2, 4, 5], 1),  # 2 .. 2,592 rows: 8 lanes
    ([2] * 8, 0), ([5] * 5, 1), ([3] * 8, 0), ([2] * 10, 0),                   # 4, 2 and 1 lanes
    ([1] * 16 + [2], 0), ([2] + [1] * 17, 1),                                  # sites >= 16
]


@pytest.mark.parametrize("cols", [1, 2, 3, 7, 16, 64])
@pytest.mark.parametrize("case", range(len(SYSTEMS)))
def test_product_matches_oracle(case, cols):
    import paper_2607_25585_amd as F
    two_s, dip = SYSTEMS[case]
    sysm = _mixed(two_s, 50 + case, bool(dip))
    ham, ref = F.Hamiltonian(sysm), of.Ham(sysm)
    if ham.dim * cols > 1 << 20:
        cols = min(cols, 3)
    ham.set_tuning(F.FTLM_C128, cols, 1)
    ham.set_tuning(F.FTLM_C64, cols, 1)
    rng = np.random.default_rng(case)
    v = rng.standard_normal((ham.dim, cols)) + 1j * rng.standard_normal((ham.dim, cols))
    want = np.stack([ref.apply(np.ascontiguousarray(v[:, c])) for c in range(cols)], 1)
    print("case", two_s, cols, flush=True)
    for dt, tol in ((torch.complex128, 1e-12), (torch.complex64, 2e-5)):
        got = ham.apply(torch.as_tensor(v if cols > 1 else v[:, 0], device="cuda").to(dt)).cpu().numpy()
        assert np.max(np.abs(got.reshape(want.shape) - want)) < tol * np.max(np.abs(want))


@pytest.mark.parametrize("columns", [1, 3, 5, 8, 12])
def test_column_sums_match_oracle(columns):
    import paper_2607_25585_amd as F
    sysm = _mixed([2, 1, 3, 2, 4], 77, True)
    T = np.array([0.5, 5.0, 50.0])
    print("case columns", columns, flush=True)
    got = F.run(F.Hamiltonian(sysm), 12, 30, T, seed=2, columns=columns)
    want = of.ftlm(sysm, 12, 30, T, seed=2)[0]
    for k in ("lnZ", "E", "C", "M"):
        d = np.max(np.abs(got[k][0] - want[k]) / np.maximum(np.abs(want[k]), 1e-3 * np.max(np.abs(want[k]))))
        assert d < 1e-8, k
