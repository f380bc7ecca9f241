"""Krylov eigenpairs of thousands of short columns, which take a lane per column: on both
sides of the number of columns and of the length where that begins, blocks that are not
full, columns cut short, matrices that split, are graded, diagonal or zero.  Every column
is, to the bit, what it is among few columns, and samples agree with NumPy."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nl,nc", [(1, 7168), (2, 7201), (10, 7167), (10, 7168), (33, 7300), (64, 7168), (100, 7169),
                                   (128, 7168), (129, 7168)])
def test_many_columns(nl, nc):
    import paper_2607_25585_amd as F
    rng = np.random.default_rng(nl)
    a, b, y = rng.standard_normal((nl, nc)), rng.random((nl, nc)) + 0.1, rng.standard_normal((nl, nc))
    kind = np.arange(nc) % 6
    b[rng.integers(0, nl, nc), np.arange(nc)] *= kind != 1          # splits
    grade = 10.0 ** -(np.arange(nl) % 12)
    a[:, kind == 2] *= grade[:, None]
    b[:, kind == 2] *= grade[:, None]
    b[:, kind == 3] = 0.0
    a[:, kind == 4], b[:, kind == 4] = 0.0, 0.0
    n_used = np.where(kind == 5, rng.integers(0, nl + 1, nc), nl).astype(np.int32)
    A, B, Y, N = (torch.as_tensor(x, device="cuda") for x in (a, b, y, n_used))
    print("case many columns", nl, nc, flush=True)
    got = F.tridiag_eigen(A, B, Y, N)
    for lo in (0, nc // 2, nc - 60):
        cut = slice(lo, lo + 60)
        few = F.tridiag_eigen(*(x[:, cut].contiguous() for x in (A, B, Y)), N[cut].contiguous())
        for g, f in zip(got, few):
            assert torch.equal(g[:, cut], f)
    eps, q1, qy = (x.cpu().numpy() for x in got)
    for c in list(range(12)) + list(range(nc - 12, nc)):
        n = int(n_used[c])
        assert not eps[n:, c].any() and not q1[n:, c].any() and not qy[n:, c].any()
        if n == 0:
            continue
        T = np.diag(a[:n, c]) + np.diag(b[:n - 1, c], 1) + np.diag(b[:n - 1, c], -1)
        lam = np.linalg.eigvalsh(T)
        assert np.max(np.abs(np.sort(eps[:n, c]) - lam)) <= 1e-13 * max(n, 8) * max(np.max(np.abs(lam)), 1e-300)
        # moments of the first row, and of it with y, whatever the order of the eigenvectors
        e1 = np.eye(n)[0]
        for p in range(3):
            Tp = np.linalg.matrix_power(T, p)
            size = max(np.max(np.abs(lam)), 1e-300) ** p * (1 + np.linalg.norm(y[:n, c]))
            assert abs(np.sum(q1[:n, c] ** 2 * eps[:n, c] ** p) - e1 @ Tp @ e1) <= 1e-12 * n * size
            assert abs(np.sum(q1[:n, c] * qy[:n, c] * eps[:n, c] ** p) - e1 @ Tp @ y[:n, c]) <= 1e-12 * n * size
