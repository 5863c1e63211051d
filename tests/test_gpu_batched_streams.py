"""The queues of a batch run side by side on streams of the handle: every queue
non-empty, two of them, or one; back to back calls on a stream of the caller,
whose inputs are produced there and consumed there without a synchronisation.
Each problem is a separate workgroup, so results are bitwise those of the same
problem solved in a batch of its own (one queue, the caller's stream only)."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (m, n, nrhs) by queue: at most 8, 12 and 20 sixteen-column tiles of [A | B].
Q1, Q2, Q3 = [(700, 100, 4), (65, 7, 2)], [(900, 180, 4)], [(1200, 250, 4), (520, 312, 8)]
MIXES = {"all": Q1 + Q2 + Q3, "two": Q1 + Q3, "middle": Q1 + Q2, "one": Q3}


@pytest.mark.parametrize("prec", ["FP64", "MIXED_FP32"])
@pytest.mark.parametrize("mix", sorted(MIXES))
def test_batched_queues_side_by_side(mix, prec):
    import paper_1805_05278_amd as m_
    h = m_.Handle(0)
    opts = h.opts(precision=getattr(m_, prec))
    probs = [(m_.to_colmajor(synth.gaussian(m, n, 70 + i)),
              m_.to_colmajor(synth.gaussian(m, k, 90 + i)))
             for i, (m, n, k) in enumerate(MIXES[mix])]
    alone = []
    for A, B in probs:
        a, b = A.clone(), B.clone()
        h.lstsq_batched([a], [b], opts)
        alone.append((a, b))
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    sums = []
    with torch.cuda.stream(s):
        for _ in range(3):
            a = [A.clone() for A, _ in probs]
            b = [B.clone() for _, B in probs]
            h.lstsq_batched(a, b, opts)
            sums.append(([x.clone() for x in a], [x.clone() for x in b]))
            for x in a + b:
                x.fill_(float("nan"))
    s.synchronize()
    for a, b in sums:
        for (ra, rb), x, y in zip(alone, a, b):
            np.testing.assert_array_equal(x.cpu().numpy(), ra.cpu().numpy())
            np.testing.assert_array_equal(y.cpu().numpy(), rb.cpu().numpy())
    h.close()


def test_server_uploads_strided_and_packed():
    """Requests whose matrices are packed or columns of a taller array, one
    column or several, in one batch: matrices and right-hand sides
    upload on a stream each."""
    import paper_1805_05278_amd as m_
    h = m_.Handle(0)
    srv = m_.Server(h, max_batch=16)
    reqs = []
    for i, (m, n, k, pad) in enumerate([(300, 40, 1, 0), (301, 41, 2, 7), (1, 1, 1, 3), (64, 1, 3, 1),
                                        (700, 130, 4, 0), (65, 9, 1, 5)]):
        A = np.asfortranarray(synth.gaussian(m + pad, n, 50 + i))[:m]
        B = np.asfortranarray(synth.gaussian(m + pad, k, 80 + i))[:m]
        X = np.zeros((n, k), order="F")
        srv.submit(A, B, X)
        reqs.append((A, B, X))
    left = len(reqs)
    while left:
        left -= len(srv.poll(wait=True))
    srv.close()
    for A, B, X in reqs:
        a, b = m_.to_colmajor(A), m_.to_colmajor(B)
        h.lstsq_batched([a], [b])
        np.testing.assert_array_equal(X, b.cpu().numpy()[:A.shape[1]])
    h.close()
