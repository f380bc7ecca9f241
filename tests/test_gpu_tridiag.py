"""Krylov eigenpairs on the GPU at the sizes and inputs where the kernels can go
wrong: around the 64 lanes of a wave, beyond the LDS (global scratch), decoupled
blocks, multiple eigenvalues (copies of a converged Ritz value), and entries of
any magnitude (the kernel scales a column by a power of two)."""
import numpy as np
import pytest
import scipy.linalg

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _columns(kind, n, rng):
    a, b = rng.standard_normal(n), np.abs(rng.standard_normal(n)) + 0.1
    if kind == "split":
        b[n // 2] = 0.0
        b[:: max(2, n // 5)] = 1e-18
    elif kind == "cluster":  # a Toeplitz block joined to its copy by a tiny element
        a[:], b[:] = 0.0, 1.0
        b[n // 2 - 1] = 1e-13
    elif kind == "zero":
        a[:], b[:] = 0.0, 0.0
    return a, b


@pytest.mark.parametrize("n", [1, 2, 3, 63, 64, 65, 129, 500, 2048, 2060])
@pytest.mark.parametrize("kind,scale", [("random", 1.0), ("split", 1.0), ("cluster", 1.0), ("random", 1e-160),
                                        ("random", 1e160), ("zero", 1.0)])
def test_eigenpairs_match_lapack(n, kind, scale):
    import paper_2607_25585_amd as F
    rng = np.random.default_rng(n)
    cols = [_columns(kind, n, rng) for _ in range(3 if n < 1000 else 1)]
    a, b = (np.stack([c[k] for c in cols], 1) for k in (0, 1))
    y = rng.standard_normal(a.shape)
    print("case", n, kind, scale, flush=True)
    dev = lambda x: torch.as_tensor(x, device="cuda")  # noqa: E731
    eps, q1, qy = [t.cpu().numpy() for t in F.tridiag_eigen(dev(a * scale), dev(b * scale), dev(y))]
    for c in range(a.shape[1]):
        ev, Q = scipy.linalg.eigh_tridiagonal(a[:, c], b[:-1, c]) if n > 1 else (a[:, c], np.ones((1, 1)))
        norm = max(np.max(np.abs(a[:, c])) + 2 * np.max(b[:, c]), 1e-300)
        # backward stable on both sides: eigenvalues to a few n eps |T|
        tol = 20 * n * 2.2e-16
        got = eps[:, c] / scale
        assert np.max(np.abs(np.sort(got) - ev)) <= tol * norm
        # the sums that the rows enter do not depend on the basis within a cluster:
        # entire functions of T, whose condition number is the exponent's range
        f, g = np.exp(-3 * (ev - ev[0]) / norm), np.exp(-3 * (got - ev[0]) / norm)
        assert abs(np.sum(q1[:, c] ** 2 * g) - np.sum(Q[0] ** 2 * f)) <= 10 * tol
        want = np.sum(Q[0] * f * (Q.T @ y[:, c]))
        assert abs(np.sum(q1[:, c] * g * qy[:, c]) - want) <= 10 * tol * np.linalg.norm(y[:, c])


@pytest.mark.parametrize("steps", [1, 2, 64, 65, 128, 140, 141])
def test_full_eigenvectors_at_their_size_limits(steps):
    # 141 steps are the most that are accepted: one rotation buffer; up to 140: two
    import ftlm_workloads as W
    import paper_2607_25585_amd as F
    from oracle import ftlm as of
    sysm, _ = W.ring_sftlm(4, 1.0)
    T = np.array([0.5, 2.0, 10.0, 60.0])
    print("case steps", steps, flush=True)
    got = F.run_sftlm(F.Hamiltonian(sysm), 2, steps, T, seed=3)
    ref = of.sftlm(sysm, 2, steps, T, seed=3)[0]
    for k in ("lnZ", "E", "C", "M"):
        d = np.abs(got[k][0] - ref[k])
        assert np.max(d / np.maximum(np.abs(ref[k]), 1e-3 * np.max(np.abs(ref[k])) + 1e-300)) < 1e-8
