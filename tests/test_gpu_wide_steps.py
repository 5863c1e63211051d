"""Look-ahead steps wider than a panel (several panels of nb factored together
and applied as one update while the trailing matrix is large): the factors are
those of the one-stream loop over single panels, which the parity tests check
against the oracle.  Two wide steps and then single panels; panel widths that
divide the wide step and that do not.  Normwise 1e-12, the G5 tolerance of V and
T; T's blocks exactly zero below their diagonals.
"""
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,nb", [(120000, 900, 64), (120000, 900, 96), (90000, 1100, 128)])
def test_wide_steps_equal_single_panels(m, n, nb):
    import paper_1805_05278_amd as miqr
    h = miqr.Handle(0)
    A0 = synth.gaussian_device(m, n, 8000 + nb)
    out = []
    for la in (True, False):
        A, T = miqr.colmajor(m, n), miqr.colmajor(nb, n)
        A.copy_(A0)
        T.fill_(3.0)
        h.factor(A, T, h.opts(t_layout=miqr.T_BLOCKED, nb=nb, lookahead=la))
        torch.cuda.synchronize()
        out.append((A, T))
    h.close()
    (Aw, Tw), (A1, T1) = out
    Rw, R1 = torch.triu(Aw[:n]), torch.triu(A1[:n])
    assert float((Rw - R1).norm() / R1.norm()) <= 1e-12
    assert float((Aw - A1).norm() / A1.norm()) <= 1e-12
    assert float((Tw - T1).norm() / T1.norm()) <= 1e-12
    rows = torch.arange(nb, device="cuda")[:, None]
    below = rows > torch.arange(n, device="cuda")[None, :] % nb
    assert bool((Tw[below.expand(nb, n)] == 0.0).all())
