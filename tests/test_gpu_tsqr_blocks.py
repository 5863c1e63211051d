"""The TSQR block factorisation at the edges of its tiles: panel widths around
multiples of 16, blocks that end inside a row tile or a row pair, 128- and
256-row leaves, chains, nodes of one child per wave and nodes whose children
are packed, panels that are not 16-byte aligned, and zero columns.  Gates:
those of the parity tests (R~ 1e-13, V and T 1e-12, normwise and by column).
"""
import numpy as np
import pytest

import oracle
import synth
from tests.test_gpu_parity import check_against_oracle, gpu_factor

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def miqr():
    import paper_1805_05278_amd as m
    h = m.Handle(0)
    yield m, h
    h.close()


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("m,tune", [
    (64, {}), (129, {}),                                # one block; an odd one
    (777, dict(leaf_rows=128, chain=1, arity=2)),       # binary tree of odd blocks
    (1500, dict(leaf_rows=256, chain=3, arity=3)),      # chains
    (2305, dict(leaf_rows=256, chain=1, arity=5)),      # four stacked children, then two levels
])
def test_tile_edges(miqr, m, n, tune):
    m_, h = miqr
    A = synth.gaussian(m, n, 7000 + 64 * m + n)
    check_against_oracle(A, gpu_factor(m_, h, A, bstar=64, b=64, **tune))


@pytest.mark.parametrize("n,arity", [(10, 17), (16, 17), (17, 16), (30, 9), (40, 7), (50, 6)])
def test_packed_children(miqr, n, arity):
    """More than four stacked children: the rows of a node lie one child after
    the other, across the row tiles."""
    m_, h = miqr
    A = synth.gaussian(128 * 20 + 5, n, 7100 + n)
    check_against_oracle(A, gpu_factor(m_, h, A, leaf_rows=128, chain=1, arity=arity))


@pytest.mark.parametrize("m,n,off", [(700, 64, 1), (1030, 37, 3), (5000, 130, 1)])
def test_unaligned_panels(miqr, m, n, off):
    """A at an odd offset and with an odd leading dimension: only 8-byte
    aligned, and its neighbours are left as they were."""
    m_, h = miqr
    A = synth.gaussian(m, n, 7200 + m)
    ld = m + off + 2 - (m + off) % 2 + 1
    big = torch.full((n + 2, ld), 7.0, dtype=torch.float64, device="cuda")
    V = big.t()[off:off + m, 1:n + 1]
    V.copy_(m_.to_colmajor(A))
    T = m_.colmajor(n, n)
    h.factor(V, T)
    torch.cuda.synchronize()
    vr = V.cpu().numpy()
    check_against_oracle(A, {"V": np.tril(vr, -1) + np.eye(m, n), "R": np.triu(vr[:n]),
                             "T": T.cpu().numpy()})
    V.fill_(7.0)
    assert bool((big == 7.0).all())


@pytest.mark.parametrize("cols", [[0], [5, 16], [63], list(range(16, 32))])
def test_zero_columns(miqr, cols):
    """Zero columns, wherever their sub-panel: no reflection, and the factors
    stay a factorisation (R is not unique there): ||A - QR|| / ||A|| <= 1e-14,
    ||Q^T Q - I|| <= 1e-13 with Q = I - V T V^T, the parity tests' gates."""
    m_, h = miqr
    A = np.asfortranarray(synth.gaussian(1500, 64, 7300))
    A[:, cols] = 0.0
    g = gpu_factor(m_, h, A)
    Q = np.eye(1500, 64) - g["V"] @ (g["T"] @ g["V"][:64].T)
    assert np.linalg.norm(A - Q @ g["R"]) <= 1e-14 * np.linalg.norm(A)
    assert np.linalg.norm(Q.T @ Q - np.eye(64)) <= 1e-13
    assert np.all(g["R"][:, cols] == 0.0)
