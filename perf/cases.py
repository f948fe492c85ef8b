"""Workloads of the block-tridiagonal Cholesky library, one pass of each through its public entry points.

A case names an entry path and its sizes: N diagonal blocks of order n, m right-hand sides, a precision
("fp64", "fp32_ir", "bf16_ir").  The matrices are the repository's synthetic recipe: D_i = G G^T / n + 4 I,
E_i ~ N(0, 1) / sqrt(n), B ~ N(0, 1), drawn on the device from the seed alone.

Paths:
  refactor_solve  an existing handle gets a new matrix (Factor.refactor) and solves with it
  solve           repeated solves with a factor that is kept
  graph           refactor + solve of one instance replayed from a recorded level schedule
  batch           factor_batched + solve_batched over many uneven instances
  served          one request of every client through the continuous-batching server
  arrow           refactor + solve of an arrow matrix (many right-hand sides: its border)
"""
import math

import torch

from paper_2601_03754_amd import btc

DEV = "cuda:0"
PRECISIONS = {"fp64": btc.BTC_FP64, "fp32_ir": btc.BTC_FP32_IR, "bf16_ir": btc.BTC_BF16_IR}
BATCH_N = (8, 16, 24, 32, 48)


def _single(name, path, N, n, m, precision, info=False):
    return {"name": name, "path": path, "N": N, "n": n, "m": m, "precision": precision, "info": info}


def listed():
    return [
        # the smallest system of the paper's setting (a short MPC horizon): launch latency
        _single("mpc_16x8", "refactor_solve", 16, 8, 1, "fp64"),
        # an MPC loop that replays its level schedule as a graph: n between padded sizes, ragged N
        _single("mpc_graph_50x12", "graph", 50, 12, 1, "fp64"),
        # the paper's block size 32 at a chain length that is no power of two
        _single("horizon_1000x32", "refactor_solve", 1000, 32, 1, "fp64"),
        # BF16 products with refinement, odd chain, block size between padded sizes, outcome wanted
        _single("bf16_511x50", "refactor_solve", 511, 50, 1, "bf16_ir", True),
        # mixed-precision solves against a kept factor, several right-hand sides
        _single("fp32_solve_4096x64x4", "solve", 4096, 64, 4, "fp32_ir"),
        # the largest served shape, FP64: a re-linearised system
        _single("refactor_4096x96", "refactor_solve", 4096, 96, 1, "fp64"),
        # the same in mixed precision, outcome wanted
        _single("fp32_refactor_4096x96", "refactor_solve", 4096, 96, 1, "fp32_ir", True),
        # the largest block size, ragged chain, an odd number of right-hand sides, kept factor
        _single("solve_1023x128x5", "solve", 1023, 128, 5, "fp64"),
        # the largest single system of the FP64 sweep
        _single("refactor_16384x128", "refactor_solve", 16384, 128, 1, "fp64"),
        # the many-instance batch of the benchmark: 512 uneven instances
        {"name": "batch_512", "path": "batch", "count": 512, "N_lo": 32, "N_hi": 2048, "precision": "fp64", "m": 1},
        # the serving loop: every client one request, three in ten with a new matrix
        {"name": "served_64", "path": "served", "count": 64, "N_lo": 64, "N_hi": 4096, "precision": "fp32_ir", "m": 1},
        # an arrow matrix: the border is solved as 40 right-hand sides, then one system
        {"name": "arrow_1000x24x40", "path": "arrow", "N": 1000, "n": 24, "border": 40, "m": 1, "precision": "fp64"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["refactor_solve"] * 4 + ["solve"] * 3 + ["graph", "batch", "served", "arrow"])
    precision = rng.choice(["fp64", "fp64", "fp32_ir", "fp32_ir", "bf16_ir"])
    m = rng.choice([1, 1, 1, 2, 3, 4, 5, 8])
    if path in ("refactor_solve", "solve"):
        c = {"path": path, "N": _log_int(rng, 16, 8192), "n": _log_int(rng, 4, 128), "m": m, "precision": precision,
             "info": rng.random() < 0.5}
        # the refinement of BF16 factors is only affordable when the caller asks for the outcome
        return dict(c, info=True) if precision == "bf16_ir" else c
    if path == "graph":
        return {"path": path, "N": _log_int(rng, 16, 512), "n": rng.randint(4, 64), "m": min(m, 4),
                "precision": rng.choice(["fp64", "fp32_ir"]), "info": False}
    if path == "batch":
        return {"path": path, "count": _log_int(rng, 24, 384), "N_lo": 32, "N_hi": _log_int(rng, 128, 2048),
                "precision": rng.choice(["fp64", "fp32_ir"]), "m": 1}
    if path == "served":
        return {"path": path, "count": rng.randint(8, 64), "N_lo": 64, "N_hi": _log_int(rng, 256, 4096),
                "precision": rng.choice(["fp64", "fp32_ir"]), "m": 1}
    return {"path": path, "N": _log_int(rng, 64, 4096), "n": rng.randint(4, 64), "border": rng.randint(2, 64),
            "m": min(m, 4), "precision": rng.choice(["fp64", "fp32_ir"])}


# ---------------------------------------------------------------------------
# inputs

def _system(g, N, n, m):
    G = torch.randn((N, n, n), generator=g, device=DEV, dtype=torch.float64)
    D = torch.bmm(G, G.transpose(1, 2).contiguous()) / n
    del G
    low = torch.tril(D)
    D = (low + torch.tril(D, -1).transpose(1, 2)).contiguous()
    D.diagonal(dim1=1, dim2=2).add_(4.0)
    E = torch.randn((N - 1, n, n), generator=g, device=DEV, dtype=torch.float64) / math.sqrt(n)
    B = torch.randn((N, n, m), generator=g, device=DEV, dtype=torch.float64)
    return D, E, B


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _shapes(case):
    """(N, n) of the instances of a batch or of the clients of a server: part of the case, not of the inputs."""
    g = torch.Generator().manual_seed(1000 + case["count"])
    u = torch.rand((case["count"], 2), generator=g, dtype=torch.float64).tolist()
    lo, hi = case["N_lo"], case["N_hi"]
    if case["path"] == "batch":
        return [(lo + int(a * (hi - lo + 1)), BATCH_N[int(b * len(BATCH_N))]) for a, b in u]
    return [(int(round(math.exp(math.log(lo) + a * math.log(hi / lo)))), 12 + int(b * 85)) for a, b in u]


def _flat_like(Bs):
    """One buffer for all solutions and a view of it for each."""
    flat = torch.empty(sum(b.numel() for b in Bs), device=DEV, dtype=torch.float64)
    views, at = [], 0
    for b in Bs:
        views.append(flat[at:at + b.numel()].view(b.shape))
        at += b.numel()
    return flat, views


def _arrow_parts(case, seed):
    g = _generator(seed)
    N, n, k = case["N"], case["n"], case["border"]
    D, E, _ = _system(g, N, n, 1)
    F = torch.randn((N * n, k), generator=g, device=DEV, dtype=torch.float64) / math.sqrt(N * n)
    H = torch.randn((k, k), generator=g, device=DEV, dtype=torch.float64)
    C = H @ H.t().contiguous() / k + 8.0 * torch.eye(k, device=DEV, dtype=torch.float64)
    B = torch.randn((N * n + k, case["m"]), generator=g, device=DEV, dtype=torch.float64)
    return D, E, F, C, B


# ---------------------------------------------------------------------------
# the passes

def prepare(case, seed):
    path, prec = case["path"], PRECISIONS[case["precision"]]
    if path in ("refactor_solve", "solve"):
        D, E, B = _system(_generator(seed), case["N"], case["n"], case["m"])
        return {"case": case, "f": btc.Factor(D, E, precision=prec), "D": D, "E": E, "B": B, "X": torch.empty_like(B)}
    if path == "graph":
        D, E, B = _system(_generator(seed), case["N"], case["n"], case["m"])
        X = torch.empty_like(B)
        r = btc.Runner()
        h = _Handle(case["N"], case["n"], prec)
        r.graph_begin()
        r.factor_batched([h.h], [D], [E])
        r.solve_batched([h.h], [B], [X])
        return {"case": case, "graph": r.graph_end(), "runner": r, "h": h, "D": D, "E": E, "B": B, "X": X}
    if path == "batch":
        g = _generator(seed)
        sys = [_system(g, N, n, case["m"]) for N, n in _shapes(case)]
        flat, Xs = _flat_like([s[2] for s in sys])
        hs = [_Handle(N, n, prec) for N, n in _shapes(case)]
        return {"case": case, "runner": btc.Runner(), "h": hs, "D": [s[0] for s in sys], "E": [s[1] for s in sys],
                "B": [s[2] for s in sys], "X": flat, "Xs": Xs}
    if path == "served":
        g = _generator(seed)
        sys = [_system(g, N, n, case["m"]) for N, n in _shapes(case)]
        flat, Xs = _flat_like([s[2] for s in sys])
        srv = btc.Server(precision=prec)
        st = {"case": case, "server": srv, "sys": sys, "X": flat, "Xs": Xs,
              "ids": [srv.add_client(N, n) for N, n in _shapes(case)]}
        _serve(st, lambda k: True)  # every client's first request brings its matrix
        return st
    if path == "arrow":
        D, E, F, C, B = _arrow_parts(case, seed)
        return {"case": case, "a": btc.Arrow(D, E, F, C, precision=prec), "D": D, "E": E, "F": F, "C": C, "B": B,
                "X": torch.empty_like(B)}
    raise ValueError("unknown path %r" % path)


class _Handle:
    """Owner of a raw handle of the batched calls."""

    def __init__(self, N, n, precision):
        self.h = btc.btc_create(N, n, precision)

    def __del__(self):
        btc.btc_destroy(self.h)


def _serve(st, refactor):
    srv = st["server"]
    for k, c in enumerate(st["ids"]):
        D, E, B = st["sys"][k]
        srv.submit(c, B, st["Xs"][k], A=(D, E) if refactor(k) else None)
    left = len(st["ids"])
    while left:
        srv.step()
        left -= len(srv.poll())


def run(st):
    case, path = st["case"], st["case"]["path"]
    if path in ("refactor_solve", "solve"):
        f = st["f"]
        if path == "refactor_solve":
            f.refactor(st["D"], st["E"])
        if case["info"]:
            X, info = f.solve(st["B"], st["X"], want_info=True)
            return {"X": X, "converged": info["converged"]}
        return f.solve(st["B"], st["X"])
    if path == "graph":
        st["graph"].launch()
        return st["X"]
    if path == "batch":
        hs = [h.h for h in st["h"]]
        st["runner"].factor_batched(hs, st["D"], st["E"])
        st["runner"].solve_batched(hs, st["B"], st["Xs"])
        return st["X"]
    if path == "served":
        _serve(st, lambda k: k % 10 in (1, 4, 8))
        return st["X"]
    if path == "arrow":
        return st["a"].refactor(st["D"], st["E"], st["F"], st["C"]).solve(st["B"], st["X"])
    raise ValueError("unknown path %r" % path)


# ---------------------------------------------------------------------------
# what a pass cannot do without

def _counts(N):
    """(coupling blocks, fill blocks) of the multi-stage factor of N blocks."""
    off = fill = 0
    s = 1
    while s <= N:
        nodes = (N + s) // (2 * s)
        right = (N - s - s) // (2 * s) + 1 if N >= 2 * s else 0  # nodes i = s(2k+1) with i + s <= N
        left = nodes - 1                                       # all but the first
        off += right + left
        fill += max(0, min(right, nodes) - 1)
        s *= 2
    return off, fill


def _work_one(N, n, m, precision, factor, solve):
    """Inputs read once, results (the kept factor among them) written once; a solve alone reads the factor once.
    Flops of the multi-stage elimination: n^3/3 per pivot, n^3 per coupling solve and its product, 2 n^3 per fill."""
    word = 8 if precision == "fp64" else 4
    tri, nn = n * (n + 1) // 2, n * n
    off, fill = _counts(N)
    A = 8 * (N * tri + (N - 1) * nn)
    L = word * (N * tri + off * nn)
    b = fl = 0
    if factor:
        b += A + L
        fl += n ** 3 * (N / 3 + 2 * off + 2 * fill)
    if solve:
        b += 16 * N * n * m + (0 if factor else L + (A if precision != "fp64" else 0))
        rounds = 1 if precision == "fp64" else 2
        fl += rounds * nn * m * (2 * N + 4 * off)
    return b, fl


def work(case):
    path, p, m = case["path"], case["precision"], case["m"]
    if path in ("refactor_solve", "graph", "solve"):
        b, f = _work_one(case["N"], case["n"], m, p, path != "solve", True)
    elif path == "arrow":
        N, n, k = case["N"], case["n"], case["border"]
        b, f = _work_one(N, n, k + m, p, True, True)
        b += 8 * (k * k + 2 * k * m)
        f += 2 * N * n * k * (k + 2 * m) + k ** 3 / 3
    else:
        b = f = 0
        for j, (N, n) in enumerate(_shapes(case)):
            x, y = _work_one(N, n, m, p, path == "batch" or j % 10 in (1, 4, 8), True)
            b, f = b + x, f + y
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# the same results from plain torch in 64 bits

def _spd_inverse(A):
    """Inverses of symmetric positive definite blocks: halves by their Schur complement, small blocks by Cholesky."""
    n = A.shape[1]
    if n <= 48:
        out = torch.empty_like(A)
        eye = torch.eye(n, device=A.device, dtype=A.dtype)
        for k in range(0, A.shape[0], 1024):
            low = torch.linalg.cholesky(A[k:k + 1024])
            inv = torch.linalg.solve_triangular(low, eye.expand_as(low).contiguous(), upper=False)
            out[k:k + 1024] = torch.bmm(inv.transpose(1, 2).contiguous(), inv)
        return out
    h = n // 2
    I11 = _spd_inverse(A[:, :h, :h].contiguous())
    W = torch.bmm(A[:, h:, :h].contiguous(), I11)
    I22 = _spd_inverse(A[:, h:, h:] - torch.bmm(W, A[:, h:, :h].transpose(1, 2).contiguous()))
    B21 = -torch.bmm(I22, W)
    B11 = I11 - torch.bmm(W.transpose(1, 2).contiguous(), B21)
    return torch.cat([torch.cat([B11, B21.transpose(1, 2)], dim=2), torch.cat([B21, I22], dim=2)], dim=1)


def _cyclic(D, E, B):
    """Solve by block cyclic reduction: the odd blocks are eliminated together, the even ones are a chain again."""
    N = D.shape[0]
    low = D[0::2]
    low = torch.tril(low) + torch.tril(low, -1).transpose(1, 2)
    inverse = _spd_inverse(low)
    n, odd = D.shape[1], inverse.shape[0]
    Lc = torch.zeros((odd, n, n), device=D.device, dtype=D.dtype)  # coupling of odd block k with the block before it
    Rc = torch.zeros_like(Lc)                                      # and (transposed) with the block after it
    Lc[1:] = E[1::2]
    Rc[:E[0::2].shape[0]] = E[0::2].transpose(1, 2)
    W = torch.bmm(inverse, torch.cat([Lc, Rc, B[0::2]], dim=2).contiguous())
    Wl, Wr, Wb = (w.contiguous() for w in (W[:, :, :n], W[:, :, n:2 * n], W[:, :, 2 * n:]))
    X = torch.empty_like(B)
    even = N // 2
    if even:
        up = Rc[:even].transpose(1, 2).contiguous()   # even block k with the odd block before it
        D2 = D[1::2] - torch.bmm(up, Wr[:even].contiguous())
        B2 = B[1::2] - torch.bmm(up, Wb[:even].contiguous())
        after = odd - 1                               # odd blocks with an even block before them
        if after:
            dn = Lc[1:].transpose(1, 2).contiguous()
            D2[:after] -= torch.bmm(dn, Wl[1:].contiguous())
            B2[:after] -= torch.bmm(dn, Wb[1:].contiguous())
        E2 = -torch.bmm(up[1:even].contiguous(), Wl[1:even].contiguous())
        X[1::2] = _cyclic(D2, E2, B2)
    x = Wb
    if even:
        x[:even] -= torch.bmm(Wr[:even].contiguous(), X[1::2].contiguous())
        if odd > 1:
            x[1:] -= torch.bmm(Wl[1:].contiguous(), X[1::2][:odd - 1].contiguous())
    X[0::2] = x
    return X


def exact(case, seed):
    path = case["path"]
    if path in ("refactor_solve", "solve", "graph"):
        X = _cyclic(*_system(_generator(seed), case["N"], case["n"], case["m"]))
        return {"X": X, "converged": None} if case["info"] and path != "graph" else X
    if path in ("batch", "served"):
        g = _generator(seed)
        return torch.cat([_cyclic(*_system(g, N, n, case["m"])).reshape(-1) for N, n in _shapes(case)])
    D, E, F, C, B = _arrow_parts(case, seed)
    N, n, k, m = case["N"], case["n"], case["border"], case["m"]
    K = N * n
    Y = _cyclic(D, E, torch.cat([F, B[:K]], dim=1).reshape(N, n, k + m).contiguous()).reshape(K, k + m)
    Z, y = Y[:, :k].contiguous(), Y[:, k:].contiguous()
    Ft = F.t().contiguous()
    tip = torch.linalg.solve(C - Ft @ Z, B[K:] - Ft @ y)
    return torch.cat([y - Z @ tip, tip], dim=0)
