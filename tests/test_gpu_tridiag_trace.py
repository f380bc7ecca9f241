"""The rotations of the tridiagonal eigensolver are orthogonal without a lean: over columns of
positive definite matrices the eigenvalues' sum keeps to the trace.  A rotation's c and s
are off by roundings of a few u = 1.1e-16; were they to one side, every rotation would
scale its rows and some 85 of them per row would move the sum by 10 u and more.  Unbiased
they move it by about sqrt(85 / steps) u, and the mean over columns by less: 4 u is the bound."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps,cols", [(60, 64), (100, 40), (100, 7168), (200, 40)])
def test_trace_is_kept(steps, cols):
    import paper_2607_25585_amd as F
    rng = np.random.default_rng(steps)
    a, b = rng.uniform(2, 4, (steps, cols)), rng.uniform(0.5, 1, (steps, cols))
    print("case trace", steps, cols, flush=True)
    eps, q1, _ = F.tridiag_eigen(torch.as_tensor(a, device="cuda"), torch.as_tensor(b, device="cuda"))
    eps, q1 = eps.cpu().numpy().astype(np.longdouble), q1.cpu().numpy().astype(np.longdouble)
    trace = a.astype(np.longdouble).sum(0)
    off = (eps.sum(0) - trace) / trace
    u = 2.0 ** -53
    assert abs(float(off.mean())) < 4 * u
    # the rows of Q stay normalised, and T_11 is what they give back
    assert abs(float((np.sum(q1 * q1, 0) - 1).mean())) < 8 * u
    assert abs(float((np.sum(q1 * q1 * eps, 0) / a[0] - 1).mean())) < 8 * u
