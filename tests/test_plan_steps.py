"""The steps of a BLOCKED factorisation as qr_plan lists them: they tile the
columns, join panels only with look-ahead, and (on the GPU) the TSQR panels that
run are those of the steps."""
import pytest

import synth


@pytest.fixture(scope="module")
def m_():
    import paper_1805_05278_amd as m
    return m


def opts(m_, nb, lookahead=True):
    return m_.Handle.opts(t_layout=m_.T_BLOCKED, nb=nb, b=64, bstar=64, lookahead=lookahead)


@pytest.mark.parametrize("m,n,nb", [(16384, 16384, 128), (8192, 8192, 96), (8000, 7777, 100),
                                    (120000, 900, 64), (12000, 9000, 16), (65536, 8192, 512),
                                    (3000, 3000, 64)])
def test_steps_tile_the_columns(m_, m, n, nb):
    for la in (True, False):
        p = m_.Handle.plan(m, n, opts(m_, nb, la))
        at, wide = 0, 0
        for c0, w in p["steps"]:
            assert c0 == at and (w == min(nb, n - c0) or w % nb == 0)
            wide = max(wide, w)
            at += w
        assert at == n
        assert (wide > nb) == (p["layout"]["tw"] > 0)
        if not la:
            assert wide == nb
    full = m_.Handle.plan(m, n, m_.Handle.opts())
    assert full["steps"] == [[0, n]]


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,nb", [(8192, 8192, 96), (120000, 700, 16), (9000, 8000, 100)])
def test_panels_run_are_the_steps_panels(m_, m, n, nb):
    torch = pytest.importorskip("torch")
    h = m_.Handle(0)
    A0 = synth.gaussian_device(m, n, 7)
    out = []
    for la in (True, False):
        o = opts(m_, nb, la)
        A, T = m_.colmajor(m, n), m_.colmajor(nb, n)
        A.copy_(A0)
        h.profile(True)
        h.factor(A, T, o)
        ran = h.profile_totals()["tsqr_hr_root"]["launches"]
        h.profile(False)
        steps = h.plan(m, n, o)["steps"]
        node = m_.Handle.opts(b=64, bstar=64)
        assert ran == sum(len(h.plan(m - c0, w, node)["panels"]) for c0, w in steps)
        out.append((A, T))
    h.close()
    # Joined or not, the same factors (the tolerance of V and T).
    for X, Y in zip(*out):
        assert float((X - Y).norm() / Y.norm()) <= 1e-12
