"""Workloads that the performance of the library is measured on.

Each case is one call (or one short sequence of calls) that a user's program
makes through ``paper_1805_05278_amd``: factorisations from 1024 x 64 to
65536 x 8192, Q applied to right-hand sides, least squares, batched small least
squares and the serving loop.  ``listed`` names the fixed cases, ``draw`` gives
more of the same ranges, ``prepare`` makes what the program has in hand before
the call, ``run`` makes the call, ``work`` counts what it cannot do without and
``exact`` is the same result from plain LAPACK-backed torch in 64 bits.

The factorisations work in place, so a program that still needs its matrix
copies it first; ``run`` does the same, which also keeps its inputs for the
next call.
"""
import torch

import paper_1805_05278_amd as miqr
import synth

_PREC = {"fp64": miqr.FP64, "fp32": miqr.MIXED_FP32, "bf16": miqr.MIXED_BF16}
_handle = None


def _h():
    """The program's handle (its workspace is kept between calls)."""
    global _handle
    if _handle is None:
        _handle = miqr.Handle(0)
    return _handle


def listed():
    return [
        # The smallest panel: one TSQR with thin Q and diag(R) >= 0, bound by
        # the latency of its launches and column steps.
        dict(name="factor_1024x64_q", kind="factor", m=1024, n=64, layout="full", q=True,
             normalize=True),
        # A small matrix of odd width: three panels of the recursion.
        dict(name="factor_600x150", kind="factor", m=600, n=150, layout="full", q=False,
             normalize=False),
        # One very tall panel with thin Q (orthogonalising a block of vectors).
        dict(name="factor_1048576x64_q", kind="factor", m=1048576, n=64, layout="full", q=True,
             normalize=False),
        # Tall and skinny over several panels with thin Q.
        dict(name="factor_262144x256_q", kind="factor", m=262144, n=256, layout="full", q=True,
             normalize=False),
        # A middling square matrix with the full kernel T of the recursion.
        dict(name="factor_4096x4096", kind="factor", m=4096, n=4096, layout="full", q=False,
             normalize=False),
        # The largest factorisations: T by panels, look-ahead on.
        dict(name="factor_16384x16384", kind="factor", m=16384, n=16384, layout="blocked",
             q=False, normalize=False),
        dict(name="factor_65536x8192", kind="factor", m=65536, n=8192, layout="blocked",
             q=False, normalize=False),
        # A kept factorisation used on new right-hand sides.
        dict(name="apply_solve_262144x256", kind="apply", m=262144, n=256, nrhs=4),
        # One large least-squares problem.
        dict(name="lstsq_65536x2048", kind="lstsq", m=65536, n=2048, nrhs=1, precision="fp64"),
        # Many small least-squares problems of the serving mix, resident in
        # device memory, in both precisions that are used for it.
        dict(name="batched_2000_fp64", kind="batched", count=2000, precision="fp64",
             m_max=4096, n_max=256),
        dict(name="batched_2000_fp32", kind="batched", count=2000, precision="fp32",
             m_max=4096, n_max=256),
        # The serving loop on host matrices: uploads, batches, solutions back.
        dict(name="server_300", kind="server", count=300, m_max=4096, n_max=256),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    """One more case: sizes spread over their logarithms, odd ones included."""
    kind = rng.choice(["factor", "factor", "factor", "factor", "apply", "lstsq", "lstsq",
                       "batched", "batched", "server"])
    if kind == "batched":
        return dict(kind=kind, count=_log_int(rng, 1, 2000),
                    precision=rng.choice(["fp64", "fp64", "fp32"]),
                    m_max=_log_int(rng, 300, 4096), n_max=_log_int(rng, 9, 256))
    if kind == "server":
        return dict(kind=kind, count=_log_int(rng, 4, 300), m_max=_log_int(rng, 300, 4096),
                    n_max=_log_int(rng, 9, 256))
    # Up to 2^27 entries and 10^12 flops.
    while True:
        n = _log_int(rng, 8, 4096)
        m = _log_int(rng, n, 1 << 20)
        if m * n <= 1 << 27 and 2.0 * m * n * n <= 1e12 and (kind == "factor" or m >= 2 * n):
            break
    if kind == "factor":
        return dict(kind=kind, m=m, n=n, layout=rng.choice(["full", "blocked"]),
                    q=rng.random() < 0.4, normalize=rng.random() < 0.3)
    if kind == "apply":
        return dict(kind=kind, m=m, n=n, nrhs=_log_int(rng, 1, 64))
    return dict(kind=kind, m=m, n=n, nrhs=rng.choice([1, 1, 2, 4, 8]),
                precision=rng.choice(["fp64", "fp64", "fp32", "bf16"]))


# ------------------------------------------------------------------ inputs

def _gaussian(m, n, seed):
    """m x n column-major N(0, 1) entries on the device."""
    return synth.gaussian_device(m, n, seed)


def _conditioned(m, n, seed, cond=100.0):
    """Gaussian columns scaled geometrically over ``cond`` and mixed by one
    reflection, so that the columns are neither orthogonal nor of one size."""
    A = _gaussian(m, n, seed)
    s = cond ** (-torch.arange(n, dtype=torch.float64, device="cuda") / max(n - 1, 1))
    A.mul_(s)
    v = _gaussian(n, 1, seed + 1)
    v.div_(v.norm())
    A.addr_((A @ v).reshape(-1), v.reshape(-1), alpha=-2.0)
    return A


def _shapes(case, seed):
    """(m, n, nrhs) of a batch's problems (the serving mix, cut to the case's
    largest sizes)."""
    tr = synth.serving_trace(case["count"], 0.0, seed, m_range=(64, case["m_max"]),
                             n_range=(8, case["n_max"]))
    return [(r.m, r.n, r.nrhs) for r in tr]


def _views(flat, shapes):
    """Column-major (r x c) views of consecutive pieces of a flat buffer."""
    out, off = [], 0
    for r, c in shapes:
        out.append(flat[off:off + r * c].view(c, r).t())
        off += r * c
    return out


def _pool(total, seed, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    return torch.randn(total, generator=g, dtype=torch.float64, device=device)


def _batch_inputs(case, seed):
    # The shapes of a case are fixed (the work of a pass does not change with
    # the seed); the values are not.
    shp = _shapes(case, 4242 + case["count"])
    a = _pool(sum(m * n for m, n, _ in shp), 2 * seed + 1)
    b = _pool(sum(m * k for m, _, k in shp), 2 * seed + 2)
    return shp, a, b


def _opts(case, h, **kw):
    return h.opts(t_layout=miqr.T_BLOCKED if case["layout"] == "blocked" else miqr.T_FULL, **kw)


# ------------------------------------------------------------ the measured work

def prepare(case, seed):
    h = _h()
    kind = case["kind"]
    if kind == "factor":
        m, n = case["m"], case["n"]
        s = dict(case=case, h=h, A0=_gaussian(m, n, seed), A=miqr.colmajor(m, n))
        s["T"] = miqr.colmajor(h.t_rows(m, n, _opts(case, h)), n)
        s["Q"] = miqr.colmajor(m, n) if case["q"] else None
        s["sign"] = (torch.empty(n, dtype=torch.float64, device="cuda")
                     if case["normalize"] else None)
        s["opts"] = _opts(case, h, normalize=case["normalize"], sign_out=s["sign"], Q=s["Q"])
        return s
    if kind == "apply":
        m, n, k = case["m"], case["n"], case["nrhs"]
        A, T = _gaussian(m, n, seed), miqr.colmajor(n, n)
        h.factor(A, T)
        return dict(case=case, h=h, A=A, T=T, C0=_gaussian(m, k, seed + 1),
                    C=miqr.colmajor(m, k))
    if kind == "lstsq":
        m, n, k = case["m"], case["n"], case["nrhs"]
        A0 = _conditioned(m, n, seed)
        B0 = miqr.colmajor(m, k)
        B0.copy_(A0 @ _gaussian(n, k, seed + 2))
        B0.add_(_gaussian(m, k, seed + 3), alpha=1e-3)
        return dict(case=case, h=h, A0=A0, B0=B0, A=miqr.colmajor(m, n), B=miqr.colmajor(m, k),
                    opts=h.opts(precision=_PREC[case["precision"]]))
    shp, a, b = _batch_inputs(case, seed)
    if kind == "batched":
        s = dict(case=case, h=h, a0=a, b0=b, a=torch.empty_like(a), b=torch.empty_like(b),
                 opts=h.opts(precision=_PREC[case["precision"]]))
        s["As"] = _views(s["a"], [(m, n) for m, n, _ in shp])
        s["Bs"] = _views(s["b"], [(m, k) for m, _, k in shp])
        return s
    # server: requests in pinned host memory, solutions into host memory
    pa = torch.empty(a.numel(), dtype=torch.float64, pin_memory=True).copy_(a)
    pb = torch.empty(b.numel(), dtype=torch.float64, pin_memory=True).copy_(b)
    x = torch.zeros(sum(n * k for _, n, k in shp), dtype=torch.float64)
    return dict(case=case, srv=miqr.Server(h, hbm_budget=1 << 30, max_batch=1024), pa=pa, pb=pb,
                x=x, As=_views(pa, [(m, n) for m, n, _ in shp]),
                Bs=_views(pb, [(m, k) for m, _, k in shp]),
                Xs=_views(x, [(n, k) for _, n, k in shp]))


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "factor":
        s["A"].copy_(s["A0"])
        s["h"].factor(s["A"], s["T"], s["opts"])
        out = {"factors": s["A"], "T": s["T"]}
        if case["q"]:
            out["Q"] = s["Q"]
        if case["normalize"]:
            out["sign"] = s["sign"]
        return out
    if kind == "apply":
        n = case["n"]
        s["C"].copy_(s["C0"])
        s["h"].apply_q("T", s["A"], s["T"], s["C"])
        s["h"].solve_r(s["A"], s["C"][:n])
        return s["C"]
    if kind == "lstsq":
        s["A"].copy_(s["A0"])
        s["B"].copy_(s["B0"])
        s["h"].lstsq(s["A"], s["B"], s["opts"])
        x = s["B"][:case["n"]]
        # A mixed factorisation leaves factors of its own precision: the
        # solution is its result.
        return {"x": x, "factors": s["A"]} if case["precision"] == "fp64" else {"x": x}
    if kind == "batched":
        s["a"].copy_(s["a0"])
        s["b"].copy_(s["b0"])
        s["h"].lstsq_batched(s["As"], s["Bs"], s["opts"])
        return {"b": s["b"], "a": s["a"]} if case["precision"] == "fp64" else {"b": s["b"]}
    left = 0
    for A, B, X in zip(s["As"], s["Bs"], s["Xs"]):
        s["srv"].submit(A, B, X)
        left += 1
    while left:
        left -= len(s["srv"].poll(wait=True))
    return s["x"]


def work(case):
    """Bytes and flops that one pass cannot do without."""
    kind = case["kind"]
    if kind in ("batched", "server"):
        by = fl = 0.0
        for m, n, k in _shapes(case, 4242 + case["count"]):
            by += 8.0 * (m * (n + k) + n * k + (n * (n + 1) / 2 if kind == "batched" else 0))
            fl += 2.0 * m * n * n - 2.0 * n ** 3 / 3.0 + 4.0 * m * n * k + 1.0 * n * n * k
        return {"bytes": by, "flops": fl}
    m, n = case["m"], case["n"]
    qr = 2.0 * m * n * n - 2.0 * n ** 3 / 3.0
    if kind == "factor":
        nq = m * n if case["q"] else 0
        return {"bytes": 8.0 * (2.0 * m * n + n * min(n, 128) / 2.0 + nq),
                "flops": qr * (2.0 if case["q"] else 1.0)}
    k = case["nrhs"]
    if kind == "apply":
        return {"bytes": 8.0 * (m * n + n * n / 2.0 + 2.0 * m * k),
                "flops": 4.0 * m * n * k + 1.0 * n * n * k}
    return {"bytes": 8.0 * (2.0 * m * n + m * k + n * k), "flops": qr + 4.0 * m * n * k}


# ------------------------------------------------------------ plain 64-bit results

def _geqrf(A):
    """(factors, tau) of LAPACK's dgeqrf (the same sign rule)."""
    a, tau = torch.geqrf(A)
    return a, tau


def _kernel_t(V, tau):
    """T of I - V T V^T from T^-1 = striu(V^T V) + diag(1 / tau); a zero tau
    leaves its row and column zero."""
    n = tau.numel()
    on = torch.nonzero(tau != 0).reshape(-1)
    Vn = V[:, on]
    G = torch.triu(Vn.t() @ Vn, 1) + torch.diag(1.0 / tau[on])
    Ti = torch.linalg.solve_triangular(G, torch.eye(on.numel(), dtype=G.dtype), upper=True)
    T = torch.zeros(n, n, dtype=V.dtype)
    T[on[:, None], on[None, :]] = Ti
    return T


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batched", "server"):
        shp, a, b = _batch_inputs(case, seed)
        a, b = a.cpu(), b.cpu()
        if sum(2.0 * m * n * n for m, n, _ in shp) > 3e11:
            return None
        As = _views(a, [(m, n) for m, n, _ in shp])
        Bs = _views(b, [(m, k) for m, _, k in shp])
        X = []
        for A, B in zip(As, Bs):
            n = A.shape[1]
            f, tau = _geqrf(A)
            c = torch.ormqr(f, tau, B, left=True, transpose=True)[:n]
            x = torch.linalg.solve_triangular(torch.triu(f[:n]), c, upper=True)
            X.append(x.t().reshape(-1))
            B[:n] = x
        if kind == "server":
            return torch.cat(X)
        # The batched sweep leaves R with row signs of its own (each row block
        # restarts the reflector's sign rule), so A has no value here.
        return {"b": b, "a": None} if case["precision"] == "fp64" else {"b": b}
    m, n = case["m"], case["n"]
    if 2.0 * m * n * n > 6e11:
        return None
    if kind == "factor":
        f, tau = _geqrf(_gaussian(m, n, seed).cpu())
        V = torch.tril(f, -1)
        V.diagonal().fill_(1.0)
        D = torch.ones(n, dtype=torch.float64)
        if case["normalize"]:
            D[torch.diagonal(f) < 0] = -1.0
        out = {}
        if case["q"]:
            out["Q"] = torch.linalg.householder_product(f, tau) * D
        if case["normalize"]:
            out["sign"] = D
            f = torch.cat([torch.tril(f[:n], -1) + D[:, None] * torch.triu(f[:n]), f[n:]])
        out["factors"] = f
        nb = _h().t_rows(m, n, _opts(case, _h()))
        T = torch.zeros(nb, n, dtype=torch.float64)
        for j in range(0, n, nb):
            w = min(nb, n - j)
            T[:w, j:j + w] = _kernel_t(V[j:, j:j + w], tau[j:j + w])
        out["T"] = T
        return out
    if kind == "apply":
        k = case["nrhs"]
        f, tau = _geqrf(_gaussian(m, n, seed).cpu())
        C = torch.ormqr(f, tau, _gaussian(m, k, seed + 1).cpu(), left=True, transpose=True)
        C[:n] = torch.linalg.solve_triangular(torch.triu(f[:n]), C[:n], upper=True)
        return C
    s = prepare(case, seed)
    A, B = s["A0"].cpu(), s["B0"].cpu()
    f, tau = _geqrf(A)
    c = torch.ormqr(f, tau, B, left=True, transpose=True)[:n]
    x = torch.linalg.solve_triangular(torch.triu(f[:n]), c, upper=True)
    return {"x": x, "factors": f} if case["precision"] == "fp64" else {"x": x}
