"""Products with few columns (right-hand sides) and the solves behind them:
Q^T C and Q C of full-T factors with 1 .. 17 columns at the edges of the thin
kernels' tiles, chunks and row split, odd leading dimensions, and R x = b at
the edges of the 64-row diagonal blocks, also with diagonals outside the range
in which a reciprocal is used."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.fixture(scope="module")
def miqr():
    import paper_1805_05278_amd as m
    h = m.Handle(0)
    yield m, h
    h.close()


def padded(m_, X, pad):
    """X on the device inside a matrix of `pad` more rows."""
    big = m_.to_colmajor(np.vstack([X, np.full((pad, X.shape[1]), np.nan)]))
    return big[:X.shape[0]]


@pytest.mark.parametrize("m,n,pad", [(1024, 64, 0), (1025, 65, 1), (1279, 16, 3), (4099, 130, 1),
                                     (65537, 40, 0), (131072 + 511, 17, 1)])
def test_thin_apply(miqr, m, n, pad):
    m_, h = miqr
    A = padded(m_, synth.gaussian(m, n, 5), pad)
    T = m_.to_colmajor(np.zeros((n, n)))
    h.factor(A, T)
    F, Th = A.cpu().numpy(), np.triu(T.cpu().numpy())
    V = np.tril(F, -1)
    V[np.arange(n), np.arange(n)] = 1.0
    for k in (1, 3, 4, 5, 8, 9, 16, 17):
        C0 = synth.gaussian(m, k, 11 + k)
        for op, Tt in (("T", Th.T), ("N", Th)):
            C = padded(m_, C0, pad)
            h.apply_q(op, A, T, C)
            ref = C0 - V @ (Tt @ (V.T @ C0))
            # Sums of m and n terms with random signs on both sides.
            assert np.linalg.norm(C.cpu().numpy() - ref) <= 40 * U * np.sqrt(m) * np.linalg.norm(C0)


@pytest.mark.parametrize("scale", [0, -1010, 1005])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 63, 64, 65, 130])
def test_thin_solve(miqr, n, scale):
    m_, h = miqr
    rng = np.random.default_rng(n)
    R = np.triu(rng.standard_normal((n, n))) / np.sqrt(n) + 2.0 * np.eye(n)
    for k in (1, 4, 5):
        b = rng.standard_normal((n, k))
        X = m_.to_colmajor(b * 2.0 ** scale)
        h.solve_r(m_.to_colmajor(R * 2.0 ** scale), X)
        x = X.cpu().numpy()
        # Componentwise backward error of a substitution: n + 1 roundings of
        # |R| |x|, and one more for a quotient that is not the nearest.
        assert (np.abs(R @ x - b) <= 2 * (n + 2) * U * (np.abs(R) @ np.abs(x))).all()
