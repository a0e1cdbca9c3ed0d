"""The work a program gives this library, as cases that can be timed and checked.

listed() names twelve cases, one for each way the library is used in earnest,
from the smallest least-squares call to the largest factorizations; draw()
gives more cases of the same kinds over their whole ranges.  prepare() makes
what the program has in hand (device matrices, options, a workspace it keeps,
a factorization or a batch plan it reuses), run() is one pass through the
public calls and returns everything they write, exact() computes the same
results with torch in 64 bits.

All inputs are column-major float64 device tensors, iid N(0, 1) unless a case
says otherwise (the paper's matrices are dense with no stated distribution),
drawn from a device generator seeded with (seed).
"""
from __future__ import annotations

import math

import torch

import paper_0912_2572_amd as tl

TREES = {"binary": tl.TREE_BINARY, "quad": tl.TREE_QUAD, "flat": tl.TREE_FLAT, "xcd": tl.TREE_XCD}


def listed():
    return [
        # one small regression: latency and launches are what counts
        {"name": "solve_small", "kind": "solve", "m": 4096, "n": 16, "k": 1, "row_block": 1024, "domains": 0,
         "tree": "binary", "q": True},
        # the serving-size call that must not allocate, on an odd shape with several right-hand sides
        {"name": "noalloc_ragged", "kind": "noalloc", "m": 50001, "n": 24, "k": 3, "row_block": 1024,
         "tree": "binary"},
        # the benchmark step: factor, thin Q and one solve of a large tall-skinny matrix
        {"name": "solve_large", "kind": "solve", "m": 1048576, "n": 64, "k": 1, "row_block": 4096, "domains": 0,
         "tree": "binary", "q": True},
        # QR of a very narrow matrix (R and Q, no solve) over load-balanced domains
        {"name": "qr_narrow", "kind": "qr", "m": 1048576, "n": 8, "row_block": 0, "domains": -1, "tree": "xcd"},
        # a kept factorization used again: new right-hand sides projected onto range(A) with Q^T and Q
        {"name": "project_rhs", "kind": "project", "m": 300001, "n": 40, "k": 24, "row_block": 4096,
         "tree": "quad"},
        # mixed precision: FP32 reflectors, refined to FP64, two panels, two right-hand sides
        {"name": "mixed_128", "kind": "mixed", "m": 524288, "n": 128, "k": 2, "row_block": 4096, "cond_exp": 2.0},
        # a wide regression: eight 64-column panels with trailing updates
        {"name": "wide_512", "kind": "solve", "m": 131072, "n": 512, "k": 1, "row_block": 0, "domains": -1,
         "tree": "binary", "q": False},
        # one block step of a block Krylov method: a new block against the basis so far
        {"name": "orth_block", "kind": "orth", "m": 1048576, "nv": 96, "b": 16, "row_block": 4096},
        # many independent regressions of mixed sizes in one graph-captured run
        {"name": "batch_64", "kind": "batch", "count": 64, "m_lo": 1000, "m_hi": 200000, "mixed": True},
        # LU of a tall panel with tournament pivoting
        {"name": "tslu_panel", "kind": "tslu", "m": 1048576, "b": 64, "row_block": 4096},
        # LU of a square matrix
        {"name": "calu_4096", "kind": "calu", "m": 4096, "n": 4096, "row_block": 256},
        # Cholesky of a Gram matrix
        {"name": "chol_8192", "kind": "chol", "n": 8192},
    ]


def _log(rng, lo, hi):
    """A whole number spread evenly over its logarithm, odd ones among them."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "noalloc", "qr", "project", "mixed", "wide", "orth", "batch", "tslu",
                       "calu", "chol"])
    tree = rng.choice(["binary", "binary", "quad", "flat", "xcd"])
    if kind in ("solve", "qr"):
        n = rng.randint(1, 64)
        m = max(_log(rng, 1000, 1048576), 4 * n)
        balanced = rng.random() < 0.3
        rb = 0 if balanced else rng.choice([512, 1024, 2048, 4096])
        if tree == "flat" and (balanced or m > 64 * rb):
            tree = "binary"     # one serial chain over hundreds of domains is nobody's choice
        c = {"kind": kind, "m": m, "n": n, "row_block": rb, "domains": -1 if balanced else 0, "tree": tree}
        if kind == "solve":
            c.update(k=rng.randint(1, 8), q=rng.random() < 0.5)
        return c
    if kind == "noalloc":
        # the static workspace is 64 MiB: about 2.5 M entries with their factors
        n = rng.randint(4, 64)
        m = _log(rng, 8 * n, 2000000 // n)
        return {"kind": kind, "m": m, "n": n, "k": rng.randint(1, 4), "row_block": 1024,
                "tree": "binary" if tree == "flat" else tree}
    if kind == "project":
        n = rng.randint(4, 64)
        return {"kind": kind, "m": _log(rng, 4000, 400000), "n": n, "k": rng.randint(1, 32),
                "row_block": rng.choice([1024, 4096]), "tree": "binary" if tree == "flat" else tree}
    if kind == "mixed":
        n = rng.randint(16, 128)
        return {"kind": kind, "m": _log(rng, 16 * n, 524288), "n": n, "k": rng.randint(1, 4),
                "row_block": rng.choice([1024, 4096]), "cond_exp": rng.choice([0.0, 1.0, 2.0])}
    if kind == "wide":
        n = rng.randint(65, 512)
        return {"kind": "solve", "m": _log(rng, 8 * n, 131072), "n": n, "k": rng.randint(1, 4),
                "row_block": 0, "domains": -1, "tree": "binary", "q": rng.random() < 0.3}
    if kind == "orth":
        b = rng.randint(4, 32)
        return {"kind": kind, "m": _log(rng, 8000, 1048576), "nv": rng.randint(1, 112), "b": b, "row_block": 4096}
    if kind == "batch":
        lo = _log(rng, 300, 20000)
        return {"kind": kind, "count": rng.randint(8, 64), "m_lo": lo, "m_hi": lo * rng.randint(2, 10),
                "mixed": rng.random() < 0.5}
    if kind == "tslu":
        b = rng.randint(8, 64)
        return {"kind": kind, "m": _log(rng, 4000, 1048576), "b": b, "row_block": rng.choice([1024, 4096])}
    if kind == "calu":
        n = _log(rng, 200, 3000)
        return {"kind": kind, "m": n + rng.choice([0, 0, rng.randint(1, 999)]), "n": n, "row_block": 256}
    return {"kind": "chol", "n": _log(rng, 100, 8000)}


# ---------------------------------------------------------------------------
# inputs (torch only)


def _batch_shapes(c, seed):
    g = torch.Generator().manual_seed(seed)
    ms = torch.randint(c["m_lo"], c["m_hi"] + 1, (c["count"],), generator=g).tolist()
    # every batch of a case has the same widths, so that its cost moves little with the seed
    return [(m, (8, 16, 32, 64)[i % 4]) for i, m in enumerate(ms)]


def _inputs(c, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def gauss(m, n):
        return torch.randn((n, m), generator=g, device="cuda", dtype=torch.float64).t()

    kind = c["kind"]
    if kind in ("solve", "noalloc", "project"):
        return gauss(c["m"], c["n"]), gauss(c["m"], c["k"])
    if kind == "qr":
        return (gauss(c["m"], c["n"]),)
    if kind == "mixed":
        # columns scaled over 10^cond_exp and mixed by a rotation
        A = gauss(c["m"], c["n"])
        s = torch.logspace(0.0, -c["cond_exp"], c["n"], device="cuda", dtype=torch.float64)
        V = torch.linalg.qr(gauss(c["n"], c["n"]).cpu())[0].cuda()
        return (V @ (A * s).t()).t(), gauss(c["m"], c["k"])
    if kind == "orth":
        return _qr64(gauss(c["m"], c["nv"]))[0], gauss(c["m"], c["b"])
    if kind == "batch":
        As = [gauss(m, n) for m, n in _batch_shapes(c, seed)]
        return As, [gauss(A.shape[0], 1).reshape(-1) for A in As]
    if kind == "tslu":
        return (gauss(c["m"], c["b"]),)
    if kind == "calu":
        return (gauss(c["m"], c["n"]),)
    G = torch.randn((c["n"], 2 * c["n"]), generator=g, device="cuda", dtype=torch.float64)
    A = (G @ G.t()) / (2 * c["n"])
    return ((0.5 * (A + A.t())).t().contiguous().t(),)


# ---------------------------------------------------------------------------
# what the program has in hand, and one pass


def prepare(case, seed):
    c, kind = case, case["kind"]
    x = _inputs(c, seed)
    s = {"case": c, "x": x}
    if kind in ("solve", "qr", "noalloc", "mixed", "project"):
        k = c.get("k", 1)
        o = tl.opts(row_block=c["row_block"], domains=c.get("domains", 0), tree=TREES[c.get("tree", "binary")],
                    prec=tl.MIXED if kind == "mixed" else tl.F64, lsq_max_rhs=max(k, 1))
        m, n = c["m"], c["n"]
        s["o"] = o
        if kind != "noalloc":
            s["work"] = torch.empty(tl.workspace_bytes(m, n, o), dtype=torch.uint8, device="cuda")
        if kind in ("qr", "noalloc") or c.get("q"):
            s["Q"] = tl.empty_colmajor(m, n)
        if kind in ("qr", "noalloc"):
            s["R"] = tl.empty_colmajor(n, n)
        if kind == "project":
            s["F"] = tl.Factors(x[0], o, work=s["work"])
            s["B"] = tl.empty_colmajor(m, k)
        else:
            s["X"] = tl.empty_colmajor(n, k)
            s["resid"] = torch.empty(k, dtype=torch.float64, device="cuda")
            s["info"] = torch.empty(1, dtype=torch.int32, device="cuda")
    elif kind == "orth":
        s["o"] = tl.opts(row_block=c["row_block"])
        s["W"] = tl.empty_colmajor(c["m"], c["b"])
        s["H"], s["R"] = tl.empty_colmajor(c["nv"], c["b"]), tl.empty_colmajor(c["b"], c["b"])
    elif kind == "batch":
        precs = [i % 2 if c["mixed"] else 0 for i in range(c["count"])]
        s["batch"] = tl.Batch(x[0], x[1], precs)
        s["stream"] = torch.cuda.Stream()
    elif kind == "tslu":
        s["o"] = tl.opts(row_block=c["row_block"])
        s["L"], s["U"] = tl.empty_colmajor(c["m"], c["b"]), tl.empty_colmajor(c["b"], c["b"])
    elif kind == "calu":
        s["o"] = tl.opts(row_block=c["row_block"])
        s["A"] = tl.empty_colmajor(c["m"], c["n"])
    else:
        s["A"] = tl.empty_colmajor(c["n"], c["n"])
    return s


def run(state):
    s = state
    x, kind = s["x"], s["case"]["kind"]
    if kind in ("solve", "mixed"):
        F, X, resid, info = tl.factor_solve(x[0], x[1], s["o"], work=s["work"], X=s["X"], resid=s["resid"],
                                            info=s["info"], Q=s.get("Q"))
        out = {"X": X, "resid": resid, "info": info}
        if kind == "solve":
            out["R"] = F.R()
            if "Q" in s:
                out["Q"] = s["Q"]
        return out
    if kind == "qr":
        F = tl.Factors(x[0], s["o"], work=s["work"])
        F.form_q(s["Q"])
        return {"R": F.R(), "Q": s["Q"]}
    if kind == "noalloc":
        X, resid, info = tl.factor_solve_noalloc(x[0], x[1], s["o"], X=s["X"], resid=s["resid"], info=s["info"],
                                                 Q=s["Q"], R=s["R"])
        return {"X": X, "resid": resid, "info": info, "Q": s["Q"], "R": s["R"]}
    if kind == "project":
        # Q [I 0; 0 0] Q^T B: the coefficients Q1^T B and the projection of B
        n, B = s["case"]["n"], s["B"]
        B.copy_(x[1])
        s["F"].apply_qt_(B)
        C = B[:n].clone()
        B[n:].zero_()
        s["F"].apply_q_(B)
        return {"coef": C, "projection": B}
    if kind == "orth":
        s["W"].copy_(x[1])      # the new block, as the operator would have written it
        W, H, R = tl.block_orth(x[0], s["W"], s["o"], H=s["H"], R=s["R"])
        return {"Q": W, "H": H, "R": R}
    if kind == "batch":
        b = s["batch"]
        s["stream"].wait_stream(torch.cuda.current_stream())
        b.run(use_graph=True, stream=s["stream"])
        torch.cuda.current_stream().wait_stream(s["stream"])
        outs = b.outs
        return {"R": torch.cat([o[0].reshape(-1) for o in outs]), "x": torch.cat([o[1] for o in outs]),
                "resid": torch.cat([o[2] for o in outs]), "info": torch.cat([o[3] for o in outs])}
    if kind == "tslu":
        ipiv, L, U, info = tl.tslu(x[0], s["o"], L=s["L"], U=s["U"])
        return {"ipiv": ipiv, "L": L, "U": U, "info": info}
    if kind == "calu":
        s["A"].copy_(x[0])      # the factorization is in place
        ipiv, info = tl.calu(s["A"], s["o"])
        return {"A": s["A"], "ipiv": ipiv, "info": info}
    s["A"].copy_(x[0])          # the factorization is in place
    info = tl.cholesky(s["A"])
    return {"A": s["A"], "info": info}


def work(case):
    c, kind = case, case["kind"]

    def qr(m, n):
        return 2.0 * m * n * n - 2.0 * n ** 3 / 3.0

    if kind in ("solve", "noalloc", "mixed"):
        m, n, k = c["m"], c["n"], c["k"]
        q = kind == "noalloc" or bool(c.get("q"))
        return {"bytes": 8.0 * (m * n * (2 if q else 1) + m * k + n * n + n * k),
                "flops": qr(m, n) * (2 if q else 1) + (4.0 * m * n + n * n) * k}
    if kind == "qr":
        m, n = c["m"], c["n"]
        return {"bytes": 8.0 * (2 * m * n + n * n), "flops": 2 * qr(m, n)}
    if kind == "project":
        m, n, k = c["m"], c["n"], c["k"]
        return {"bytes": 8.0 * (m * n + 2 * m * k + n * k), "flops": 8.0 * m * n * k}
    if kind == "orth":
        m, nv, b = c["m"], c["nv"], c["b"]
        return {"bytes": 8.0 * (m * nv + 2 * m * b + nv * b + b * b), "flops": 8.0 * m * nv * b + 2 * qr(m, b)}
    if kind == "batch":
        mid = 0.5 * (c["m_lo"] + c["m_hi"])
        ns = [(8, 16, 32, 64)[i % 4] for i in range(c["count"])]
        return {"bytes": sum(8.0 * (mid * n + mid + n * n + n) for n in ns),
                "flops": sum(qr(mid, n) + 4.0 * mid * n + n * n for n in ns)}
    if kind == "tslu":
        m, b = c["m"], c["b"]
        return {"bytes": 8.0 * (2 * m * b + b * b + b), "flops": m * b * b - b ** 3 / 3.0}
    if kind == "calu":
        m, n = c["m"], c["n"]
        return {"bytes": 8.0 * (2 * m * n + n), "flops": 1.0 * m * n * n - n ** 3 / 3.0}
    n = c["n"]
    return {"bytes": 8.0 * n * n, "flops": n ** 3 / 3.0}   # the lower triangle, read and written


# ---------------------------------------------------------------------------
# the same results in 64 bits with torch


def _chol_and_inverse(A):
    """R with R^T R = A^T A and its inverse, the small matrices on the host."""
    R = torch.linalg.cholesky((A.t() @ A).cpu()).t().contiguous()
    inv = torch.linalg.solve_triangular(R, torch.eye(R.shape[0], dtype=R.dtype), upper=True)
    return R.to(A.device), inv.to(A.device)


def _qr64(A):
    """Thin QR with a positive diagonal: two Cholesky QR passes, accurate to
    rounding for the condition numbers of these cases (at most 1e2 times a
    Gaussian's)."""
    R1, inv = _chol_and_inverse(A)
    Q = A @ inv
    R2, inv = _chol_and_inverse(Q)
    Q = Q @ inv
    return Q.t().contiguous().t(), R2 @ R1


def _lsq64(A, B):
    Q, R = _qr64(A)

    def back(C):
        return torch.linalg.solve_triangular(R.cpu(), C.cpu(), upper=True).to(C.device)

    X = back(Q.t() @ B)
    X = X + back(Q.t() @ (B - A @ X))     # one step of refinement on the residual
    return Q, R, X, torch.linalg.norm(B - A @ X, dim=0)


def _pivot_rows(rows, idx, b):
    """The first b pivot rows (of A, as indices) of partial pivoting on a stack."""
    LU, piv = torch.linalg.lu_factor(rows)
    perm = idx.clone()
    for i, p in enumerate((piv[:b] - 1).tolist()):
        if p != i:
            t = perm[i].item()
            perm[i] = perm[p]
            perm[p] = t
    return perm[:b]


def _tournament(A, b, mb):
    """Pivot rows of a panel (host tensor) by tournament: domains of mb rows
    (a last one shorter than b joins its neighbour), each reduced in stacks
    of at most 256 rows, then a binary tree of adjacent pairs."""
    m = A.shape[0]
    starts = list(range(0, m, mb))
    if len(starts) > 1 and m - starts[-1] < b:
        starts.pop()
    nodes = []
    for s, e in zip(starts, starts[1:] + [m]):
        cand, pos = torch.empty(0, dtype=torch.int64), s
        while pos < e:
            take = min(e - pos, 256 - len(cand))
            idx = torch.cat([cand, torch.arange(pos, pos + take)])
            cand = _pivot_rows(A[idx, :b], idx, min(b, len(idx)))
            pos += take
        nodes.append(cand)
    while len(nodes) > 1:
        up = []
        for i in range(0, len(nodes) - 1, 2):
            idx = torch.cat([nodes[i], nodes[i + 1]])
            up.append(_pivot_rows(A[idx, :b], idx, b))
        nodes = up + (nodes[-1:] if len(nodes) % 2 else [])
    return nodes[0]


def _lu_no_pivot(P):
    """Unit lower L and U of a small square matrix whose rows are in pivot order."""
    P = P.clone()
    for j in range(P.shape[1]):
        P[j + 1:, j] /= P[j, j]
        P[j + 1:, j + 1:] -= P[j + 1:, j:j + 1] * P[j:j + 1, j + 1:]
    return torch.tril(P, -1) + torch.eye(P.shape[0], dtype=P.dtype), torch.triu(P)


def _calu64(A, mb):
    m, n = A.shape
    A = A.clone()
    for k in range(0, n, 64):
        b = min(64, n - k)
        rows = _tournament(A[k:, k:k + b].contiguous(), b, mb)
        at = torch.arange(m - k)
        for i, r in enumerate(rows.tolist()):
            p = int((at == r).nonzero()[0])
            at[[i, p]] = at[[p, i]]
        A[k:] = A[k:][at]
        L11, U11 = _lu_no_pivot(A[k:k + b, k:k + b])
        A[k:k + b, k:k + b] = torch.tril(L11, -1) + U11
        if k + b < m:
            A[k + b:, k:k + b] = torch.linalg.solve_triangular(U11, A[k + b:, k:k + b], upper=True, left=False)
        if k + b < n:
            A[k:k + b, k + b:] = torch.linalg.solve_triangular(L11, A[k:k + b, k + b:], upper=False)
            if k + b < m:
                A[k + b:, k + b:] -= A[k + b:, k:k + b] @ A[k:k + b, k + b:]
    return A


def exact(case, seed):
    c, kind = case, case["kind"]
    x = _inputs(c, seed)
    if kind in ("solve", "mixed", "noalloc"):
        Q, R, X, resid = _lsq64(*x)
        out = {"X": X, "resid": resid, "info": None}
        if kind != "mixed":
            out["R"] = R
        if kind == "noalloc" or c.get("q"):
            out["Q"] = Q
        return out
    if kind == "qr":
        Q, R = _qr64(x[0])
        return {"R": R, "Q": Q}
    if kind == "project":
        Q, _ = _qr64(x[0])
        C = Q.t() @ x[1]
        return {"coef": C, "projection": Q @ C}
    if kind == "orth":
        V, W = x
        H = V.t() @ W
        W = W - V @ H
        H2 = V.t() @ W
        Q, R = _qr64(W - V @ H2)
        return {"Q": Q, "H": H + H2, "R": R}
    if kind == "batch":
        Rs, xs, rs = [], [], []
        for A, b in zip(*x):
            _, R, X, resid = _lsq64(A, b.reshape(-1, 1))
            Rs.append(R.t().reshape(-1))     # column-major, as the library lays it out
            xs.append(X[:, 0])
            rs.append(resid)
        return {"R": torch.cat(Rs), "x": torch.cat(xs), "resid": torch.cat(rs), "info": None}
    if kind == "tslu":
        A = x[0].cpu()
        rows = _tournament(A, c["b"], c["row_block"])
        L11, U = _lu_no_pivot(A[rows])
        L = torch.linalg.solve_triangular(U, A, upper=True, left=False)
        L[rows] = L11
        return {"ipiv": None, "L": L, "U": U, "info": None}
    if kind == "calu":
        return {"A": _calu64(x[0].cpu().contiguous(), c["row_block"]), "ipiv": None, "info": None}
    A = x[0].cpu()
    return {"A": torch.tril(torch.linalg.cholesky(A)) + torch.triu(A, 1), "info": None}
