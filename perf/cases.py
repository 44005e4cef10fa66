"""Workloads that users of this library run, as timing cases.

Every case is one call sequence of a user's program through the public binding
(paper_2601_21990_amd.pdlpb, paper_2601_21990_amd.serve): a batch is set, solved
and its results are read.  Contexts (one per constraint matrix) are made
beforehand, as a branch-and-bound code keeps them between calls.

Inputs are random LPs made from the seed, of the families of workloads/: a sparse
matrix with k nonzeros per column, rows of mixed sense, a finite box.  They
are planted: a primal-dual optimum (x*, y*) is drawn first and the objective and
right-hand side follow from it, so a branching batch has its root solution to
warm-start from without a solve.

`exact` runs the same method (restarted, reflected-Halpern PDHG; arXiv
2601.21990, Sections 4 and 5) in float64 with plain torch on whole blocks.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2601_21990_amd.pdlpb as P
from paper_2601_21990_amd.serve import Request, Server

DEVICE_BYTES = 64e6      # results beyond this stay on the device
BOX = {"branch": 10.0, "tighten": 5.0, "single": 10.0, "cover": 1.0, "serve": 10.0}


def listed():
    return [
        # one small LP from a cold start to a tight tolerance: the root of a small
        # problem, or a host code that solves LPs one at a time
        {"name": "single_50x100", "kind": "single", "m": 50, "n": 100, "k": 3, "B": 1,
         "prec": "fp64", "C": 64, "S": 0, "tol": 1e-6, "iters": 3000},
        # the root LP of a middling problem
        {"name": "single_2000x5000", "kind": "single", "m": 2000, "n": 5000, "k": 5, "B": 1,
         "prec": "fp64", "C": 64, "S": 0, "tol": 1e-6, "iters": 3000},
        # the root LP of a large one (the vectors of one LP are contiguous)
        {"name": "single_200kx500k", "kind": "single", "m": 200000, "n": 500000, "k": 4, "B": 1,
         "prec": "fp64", "C": 64, "S": 0, "tol": 1e-4, "iters": 1000},
        # full strong branching at a node of a small problem, host arrays in and out
        {"name": "branch_200x500_b16", "kind": "branch", "m": 200, "n": 500, "k": 5, "B": 16,
         "prec": "fp64", "C": 32, "S": 0, "tol": 1e-4, "iters": 2000},
        # the small strong-branching batch of the benchmark
        {"name": "branch_2000x5000_b64", "kind": "branch", "m": 2000, "n": 5000, "k": 5, "B": 64,
         "prec": "fp64", "C": 32, "S": 0, "tol": 1e-4, "iters": 2000},
        # odd sizes throughout, with stopping tests between the evaluations
        {"name": "branch_12011x30011_b151", "kind": "branch", "m": 12011, "n": 30011, "k": 6,
         "B": 151, "prec": "fp64", "C": 24, "S": 12, "tol": 1e-4, "iters": 2000},
        # the benchmark line: strong branching on the largest single-GPU shape
        {"name": "branch_200kx500k_b512", "kind": "branch", "m": 200000, "n": 500000, "k": 4,
         "B": 512, "prec": "fp64", "C": 18, "S": 6, "tol": 1e-4, "iters": 2000},
        # bound tightening (+-e_j objectives, cold start) in both precisions
        {"name": "tighten_20kx50k_b256_fp32", "kind": "tighten", "m": 20000, "n": 50000, "k": 8,
         "B": 256, "prec": "fp32", "C": 64, "S": 0, "tol": 1e-4, "iters": 321},
        {"name": "tighten_20kx50k_b256", "kind": "tighten", "m": 20000, "n": 50000, "k": 8,
         "B": 256, "prec": "fp64", "C": 64, "S": 0, "tol": 1e-4, "iters": 321},
        # bound tightening up to an iteration limit on the largest shape (every LP
        # runs to the limit)
        {"name": "tighten_200kx500k_b512", "kind": "tighten", "m": 200000, "n": 500000, "k": 4,
         "B": 512, "prec": "fp64", "C": 64, "S": 0, "tol": 0.0, "iters": 65},
        # a 0/1 relaxation (set covering) with diagonal scaling and the stricter
        # dual test of the bound-tightening experiments
        {"name": "cover_2000x4000_b64", "kind": "cover", "m": 2000, "n": 4000, "k": 8, "B": 64,
         "prec": "fp64", "C": 64, "S": 0, "tol": 1e-4, "iters": 1000},
        # continuous batching: requests of mixed kinds and sizes over three resident
        # bases, admitted as columns free up, until all have finished
        {"name": "serve_3_bases", "kind": "serve", "m": 1000, "n": 2500, "k": 6, "B": 640,
         "prec": "fp64", "C": 8, "S": 0, "tol": 1e-4, "iters": 600},
    ]


def _logu(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over the listed ranges, half of them odd, batches no
    wider than the memory traffic of the largest listed case allows."""
    kind = rng.choice(["single", "branch", "branch", "tighten", "tighten", "cover", "serve"])
    prec = rng.choice(["fp64", "fp64", "fp32"]) if kind in ("tighten", "serve") else "fp64"
    m = _logu(rng, 100, {"cover": 8000, "serve": 4000}.get(kind, 200000))
    n = int(m * rng.uniform(1.6, 3.0))
    k = rng.choice([4, 5, 6, 8])
    c = {"kind": kind, "m": m, "n": n, "k": k, "prec": prec, "S": 0, "tol": 1e-4}
    if kind == "single":
        c |= {"B": 1, "C": 64, "iters": 1000}
    elif kind == "branch":
        C = rng.choice([18, 24, 32, 64])
        c |= {"B": _logu(rng, 2, 512), "C": C, "S": rng.choice([0, C // 2]), "iters": 1000}
    elif kind == "tighten":
        # the iteration budget follows the size, as the whole batch runs to it
        B = _logu(rng, 4, 512)
        c |= {"B": B, "C": 64, "iters": 321 if n * B < 20e6 else 65}
    elif kind == "cover":
        c |= {"n": 2 * m + m % 3, "B": _logu(rng, 4, 128), "C": 64, "iters": 1000}
    else:
        c |= {"B": _logu(rng, 64, 640), "C": rng.choice([8, 12, 16]), "iters": 600}
    return c


# ---- inputs ---------------------------------------------------------------------

def _csr(m, rows, cols, vals):
    """Triplets to CSR with column indices ascending in every row."""
    order = np.lexsort((cols, rows)) if rows.size < 400000 else \
        torch.sort(torch.from_numpy(rows * (int(cols.max()) + 1) + cols).cuda())[1].cpu().numpy()
    rp = np.zeros(m + 1, dtype=np.int64)
    np.cumsum(np.bincount(rows, minlength=m), out=rp[1:])
    return rp, cols[order].astype(np.int32), np.ascontiguousarray(vals[order])


def _columns(rng, m, n, k):
    """k distinct rows for every column."""
    draw = np.sort(rng.integers(0, m, size=(n, k)), axis=1)
    while True:
        bad = np.nonzero((draw[:, 1:] == draw[:, :-1]).any(axis=1))[0]
        if not bad.size:
            return draw.ravel(), np.repeat(np.arange(n), k)
        draw[bad] = np.sort(rng.integers(0, m, size=(bad.size, k)), axis=1)


def _instance(kind, m, n, k, rng):
    """A base LP as a dict, with its planted optimum x, y."""
    if kind == "cover":
        # every row covered by k columns; x = 1 is feasible
        cols, rows = _columns(rng, n, m, k)
        rp, ci, v = _csr(m, rows, cols, np.ones(m * k))
        return dict(m=m, n=n, rp=rp, ci=ci, v=v, c=rng.integers(1, 101, n).astype(np.float64),
                    b=np.ones(m), sense=np.full(m, ord("G"), np.uint8), lo=np.zeros(n), hi=np.ones(n))
    hi = BOX[kind]
    rows, cols = _columns(rng, m, n, min(k, m))
    vals = rng.uniform(-1.0, 1.0, rows.size) if kind == "tighten" else rng.standard_normal(rows.size)
    rp, ci, v = _csr(m, rows, cols, vals)
    sense = np.array([ord("E"), ord("L"), ord("G")], np.uint8)[rng.integers(0, 3, m)]
    # the optimum: a quarter of the variables strictly inside the box, the others at a
    # bound; equality rows and half of the others tight
    inside = rng.random(n) < 0.25
    at_hi = rng.random(n) < 0.5
    x = np.where(inside, rng.uniform(0.1 * hi, 0.9 * hi, n), np.where(at_hi, hi, 0.0))
    r = np.where(inside, 0.0, np.abs(rng.standard_normal(n)) * np.where(at_hi, 1.0, -1.0))
    tight = (sense == ord("E")) | (rng.random(m) < 0.5)
    y = np.where(tight, rng.standard_normal(m), 0.0)
    y = np.where(sense == ord("L"), np.abs(y), np.where(sense == ord("G"), -np.abs(y), y))
    ax = np.bincount(rows, weights=vals * x[cols], minlength=m)
    slack = np.where(tight, 0.0, rng.uniform(0.0, 1.0, m))
    b = ax + np.where(sense == ord("L"), slack, np.where(sense == ord("G"), -slack, 0.0))
    c = -np.bincount(cols, weights=vals * y[rows], minlength=n) - r
    return dict(m=m, n=n, rp=rp, ci=ci, v=v, c=c, b=b, sense=sense, lo=np.zeros(n),
                hi=np.full(n, hi), x=x, y=y, inside=np.nonzero(inside)[0])


def _branches(inst, B, rng):
    """ceil(B / 2) variables inside the box, one branch up and one down each
    (Section 5.1 order), the last one dropped when B is odd."""
    p = min((B + 1) // 2, inst["inside"].size)
    var = np.sort(rng.choice(inst["inside"], p, replace=False)).astype(np.int32)
    xv = inst["x"][var]
    D = P.deltas_array([P.SET_LO] * p + [P.SET_HI] * p, np.concatenate([var, var]),
                       np.concatenate([np.floor(xv) + 1.0, np.floor(xv)]))
    return D[:B]


def _tightenings(n, B, rng):
    """min and max of ceil(B / 2) variables (Section 5.2 order)."""
    p = min((B + 1) // 2, n)
    var = np.sort(rng.choice(n, p, replace=False)).astype(np.int32)
    return P.deltas_array([P.OBJ_UNIT] * (2 * p), np.concatenate([var, var]),
                          np.concatenate([np.ones(p), -np.ones(p)]))[:B]


def _weight(inst):
    return float(np.linalg.norm(inst["y"]) / np.linalg.norm(inst["x"])) or 1.0


def _inputs(case, seed):
    """The bases of a case and what is asked of each: (instance, changes, warm)."""
    rng = np.random.default_rng([2601021990, int(seed)])
    kind, B = case["kind"], case["B"]
    if kind == "serve":
        bases = [_instance(kind, f * case["m"] + i, f * case["n"] + 3 * i, case["k"], rng)
                 for i, f in enumerate((1, 3, 10))]
        reqs, left = [], B
        while left > 0:      # even request sizes, log-uniform in 2 ... 128
            size = min(2 * max(1, round(math.exp(rng.uniform(0.0, math.log(64.0))))), left)
            b = int(rng.integers(0, 3))
            reqs.append((b, _branches(bases[b], size, rng) if rng.random() < 0.5
                         else _tightenings(bases[b]["n"], size, rng)))
            left -= size
        return bases, reqs
    inst = _instance(kind, case["m"], case["n"], case["k"], rng)
    if kind == "single":
        return inst, P.deltas_array([P.BASE], [0], [0.0])
    return inst, _branches(inst, B, rng) if kind == "branch" else _tightenings(inst["n"], B, rng)


def _options(case):
    return dict(precision=P.MIXED32 if case["prec"] == "fp32" else P.FP64, eval_every=case["C"],
                stop_every=case["S"], scaling=1 if case["kind"] == "cover" else 0,
                dual_tol=1e-8 if case["kind"] == "cover" else -1.0)


def _context(inst, **kw):
    return P.Context(inst["m"], inst["n"], inst["rp"], inst["ci"], inst["v"], inst["c"], inst["b"],
                     inst["sense"], inst["lo"], inst["hi"], **kw)


def prepare(case, seed):
    if case["kind"] == "serve":
        bases, reqs = _inputs(case, seed)
        ctxs = []
        for inst in bases:
            ctx = _context(inst, max_batch=256, **_options(case))
            ctx.set_base_warm(inst["x"], inst["y"], _weight(inst))
            ctx.serve_begin(1024)
            ctxs.append(ctx)
        return {"case": case, "ctxs": ctxs, "reqs": reqs}
    inst, D = _inputs(case, seed)
    B = len(D)
    ctx = _context(inst, max_batch=B, **_options(case))
    st = {"case": case, "ctx": ctx, "D": D, "warm": {}, "mem": P.MEM_HOST, "out": {}}
    w = None
    if case["kind"] == "branch":
        w = np.full(B, _weight(inst))
        st["warm"] = dict(x_warm=inst["x"], y_warm=inst["y"], w_warm=w)
    if 8.0 * B * (inst["m"] + inst["n"]) > DEVICE_BYTES:
        # large batches: changes, warm start and results in device memory
        dev = torch.device("cuda", 0)
        st["mem"] = P.MEM_DEVICE
        st["D"] = torch.from_numpy(D.view(np.uint8).copy()).to(dev)
        st["warm"] = {k: torch.from_numpy(np.ascontiguousarray(v)).to(dev) for k, v in st["warm"].items()}
        st["out"] = {"X": torch.empty(B, inst["n"], dtype=torch.float64, device=dev),
                     "Y": torch.empty(B, inst["m"], dtype=torch.float64, device=dev)}
        if case["prec"] == "fp64" and case["kind"] != "cover":
            ctx.set_result_buffers(st["out"]["X"], st["out"]["Y"], B)
    return st


def run(st):
    case = st["case"]
    if case["kind"] == "serve":
        srv = Server(st["ctxs"])
        reqs = [Request(base=b, deltas=D, arrival=0.0, tol=case["tol"], max_iters=case["iters"])
                for b, D in st["reqs"]]
        for r in reqs:
            srv.submit(r)
        srv.drain()
        return {key: np.array([getattr(r, key)[i] for r in reqs for i in r.ids])
                for key in ("statuses", "iters", "objs")}
    ctx = st["ctx"]
    ctx.set_batch(st["D"], mem=st["mem"], **st["warm"])
    ctx.solve(tol=case["tol"], max_iters=case["iters"])
    return ctx.get_batch(mem=st["mem"], **st["out"])


def work(case):
    """What a pass cannot do without.  Flops: two products per iteration, with a
    nominal count of iterations per LP (half of a branching batch stops at its first
    evaluation).  Bytes: the matrix and its transpose, the results, and per
    iteration one read and one write of the iterates where they exceed the caches."""
    m, n, k, B = case["m"], case["n"], case["k"], case["B"]
    if case["kind"] == "serve":
        m, n = 14 * m // 3, 14 * n // 3
    s = 4.0 if case["prec"] == "fp32" else 8.0
    nnz = (m if case["kind"] == "cover" else n) * k
    per_lp = {"single": 600, "branch": 6 if m > 50000 else 100, "tighten": min(case["iters"], 257), "cover": 130,
              "serve": 60}[case["kind"]]
    # (served LPs run a few at a time on each base: their iterates stay in the caches)
    large = case["kind"] != "serve" and 4 * s * B * (m + n) > 256e6
    sweeps = per_lp * B * s * (4.0 * m + 4.0 * n) if large else 0.0
    out = 12.0 * B if case["kind"] == "serve" else 8.0 * B * (m + n)
    return {"bytes": 2.0 * nnz * (s + 4) + out + sweeps, "flops": 4.0 * nnz * B * per_lp}


# ---- the method in float64 with plain torch -----------------------------------------

def _scaling(inst):
    """Ten Ruiz passes (square roots of the row and column maxima), then one
    Pock-Chambolle pass (square roots of the row and column sums)."""
    m, n = inst["m"], inst["n"]
    rows, cols, v = np.repeat(np.arange(m), np.diff(inst["rp"])), inst["ci"], np.abs(inst["v"])
    dr, dc = np.ones(m), np.ones(n)
    for it in range(11):
        a = dr[rows] * v * dc[cols]
        rs, cs = np.zeros(m), np.zeros(n)
        if it < 10:
            np.maximum.at(rs, rows, a)
            np.maximum.at(cs, cols, a)
        else:
            rs, cs = np.bincount(rows, a, m), np.bincount(cols, a, n)
        dr, dc = dr / np.sqrt(np.where(rs > 0, rs, 1.0)), dc / np.sqrt(np.where(cs > 0, cs, 1.0))
    return dr, dc


def _reference(inst, D, x0, y0, w0, C, S, tol, dual_tol, iters, scaling):
    """Every LP of the batch by blocks of columns; the box is finite, so the reduced
    cost is -c - A'y whole.  Returns what get_batch does."""
    dev, f8 = torch.device("cuda", 0), torch.float64
    m, n, B = inst["m"], inst["n"], len(D)
    dr, dc = _scaling(inst) if scaling else (np.ones(m), np.ones(n))
    rows = np.repeat(np.arange(m), np.diff(inst["rp"]))
    vals = dr[rows] * inst["v"] * dc[inst["ci"]]
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    A = torch.sparse_csr_tensor(t(inst["rp"]), t(inst["ci"].astype(np.int64)), t(vals), (m, n))
    order = np.lexsort((rows, inst["ci"]))
    tp = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(inst["ci"], minlength=n), out=tp[1:])
    At = torch.sparse_csr_tensor(t(tp), t(rows[order]), t(vals[order]), (n, m))
    c, b = inst["c"] * dc, inst["b"] * dr
    sense = inst["sense"]
    lo, hi = t(inst["lo"] / dc)[:, None], t(inst["hi"] / dc)[:, None]
    rl = t(np.where(sense == ord("L"), -np.inf, b))[:, None]
    ru = t(np.where(sense == ord("G"), np.inf, b))[:, None]
    is_l, is_g = t(sense == ord("L"))[:, None], t(sense == ord("G"))[:, None]
    # step size: power iteration on A'A
    v = 1.0 + np.modf(np.arange(n) * 0.6180339887498949)[0]
    v, old, lam = t(v / np.linalg.norm(v))[:, None], 0.0, 1.0
    for _ in range(10000):
        v = At @ (A @ v)
        lam = float(v.norm())
        v = v / lam
        if abs(lam - old) <= 1e-14 * lam:
            break
        old = lam
    eta = 0.998 / math.sqrt(lam)
    # per-LP data of the LPs still running (columns)
    kind, var = D["kind"], D["var"].astype(np.int64)
    val = np.where(kind == P.OBJ_UNIT, D["value"] * dc[var], D["value"] / dc[var])
    if w0 is None:
        cn = np.where(kind == P.OBJ_UNIT, np.abs(val), np.linalg.norm(c))
        w0 = cn / np.linalg.norm(b)
    live, var, val, w = torch.arange(B, device=dev), t(var), t(val), t(w0)
    up, dn, ob = t(kind == P.SET_LO), t(kind == P.SET_HI), t(kind == P.OBJ_UNIT)
    lo_j = torch.where(up, val, lo[var, 0])
    hi_j = torch.where(dn, val, hi[var, 0])

    def project(Z):
        """Onto each LP's box, with its own bounds at its variable."""
        j = torch.arange(Z.shape[1], device=dev)
        own = Z[var, j]
        Z = torch.minimum(torch.maximum(Z, lo), hi)
        Z[var, j] = torch.where(ob, Z[var, j], torch.minimum(torch.maximum(own, lo_j), hi_j))
        return Z

    def objective(v=None):
        """c of every LP as a block (n x live)."""
        Z = t(c)[:, None] * (~ob)
        j = torch.arange(Z.shape[1], device=dev)
        Z[var, j] += torch.where(ob, val, torch.zeros_like(val))
        return Z

    support_y = lambda y: (torch.where(y > 0, ru * y, 0.0) + torch.where(y < 0, rl * y, 0.0)).sum(0)  # noqa: E731
    dots = lambda a, b_: (a * b_).sum(0)  # noqa: E731

    def support_x(r):
        j = torch.arange(r.shape[1], device=dev)
        z = torch.where(r > 0, hi * r, lo * r)
        rv = r[var, j]
        own = torch.where(rv > 0, hi_j * rv, lo_j * rv)
        return z.sum(0) - z[var, j] + own

    X = project((t(x0)[:, None] if x0 is not None else torch.zeros(n, 1, dtype=f8, device=dev)).repeat(1, B))
    Y = (t(y0)[:, None] if y0 is not None else torch.zeros(m, 1, dtype=f8, device=dev)).repeat(1, B)
    XA, YA = X, Y
    cost = objective()
    k = torch.zeros(B, dtype=f8, device=dev)
    r0, rp = torch.zeros(B, dtype=f8, device=dev), torch.full((B,), -1.0, dtype=f8, device=dev)
    X_out, Y_out = torch.zeros(B, n, dtype=f8, device=dev), torch.zeros(B, m, dtype=f8, device=dev)
    status, its = np.zeros(B, np.int32), np.zeros(B, np.int64)
    kkt, obj = np.full((B, 4), np.nan), np.full(B, np.nan)
    dtol = tol if dual_tol < 0 else dual_tol
    for it in range(iters):
        full, stop, last = it % C == 0, S and it % S == 0, it + 1 >= iters
        tau, sg = eta / w, eta * w
        XT = project(X - tau * (cost + At @ Y))
        Q = Y / sg + A @ (2.0 * XT - X)
        YT = sg * (Q - torch.minimum(torch.maximum(Q, rl), ru))
        fresh = bool((k == 0).any())
        done = torch.zeros(live.numel(), dtype=torch.int32, device=dev)
        if full or fresh:
            dX, dY = XT - X, YT - Y
            adx = A @ dX
            r = ((w / eta) * dots(dX, dX) + dots(dY, dY) / (eta * w) - 2.0 * dots(dY, adx)).clamp_min(0).sqrt()
        if full or stop or last:
            g = At @ YT
            red = -cost - g
            cx, phi = dots(cost, XT), support_x(red) + support_y(YT)
            ax = A @ XT
            pri = (ax - torch.minimum(torch.maximum(ax, rl), ru)).norm(dim=0) / (1.0 + ax.norm(dim=0))
            gap = (cx + phi).abs() / (1.0 + cx.abs() + phi.abs())
            dua = (cost + g + red).norm(dim=0) / (1.0 + cost.norm(dim=0))
            rel = torch.maximum(gap, torch.maximum(pri, dua))
            if full or stop:
                done[(gap <= tol) & (pri <= tol) & (dua <= dtol)] = P.STATUS_OPTIMAL
            if full and tol > 0.0:
                yb = torch.where(is_l, dY.clamp_min(0), torch.where(is_g, dY.clamp_max(0), dY))
                dr_ = -(At @ dY)
                ph = support_y(yb) + support_x(dr_)
                pinf = (ph < 0) & ((At @ yb + dr_).norm(dim=0) <= tol * ph.abs())
                cdx = dots(cost, dX)
                rec = torch.where(is_l, adx.clamp_max(0), torch.where(is_g, adx.clamp_min(0), torch.zeros_like(adx)))
                dinf = (cdx < 0) & (dX.norm(dim=0) <= tol * cdx.abs()) & ((adx - rec).norm(dim=0) <= tol * cdx.abs())
                done = torch.where((done == 0) & pinf, P.STATUS_PRIMAL_INFEASIBLE, done)
                done = torch.where((done == 0) & dinf, P.STATUS_DUAL_INFEASIBLE, done)
            if last:
                done = torch.where(done == 0, P.STATUS_ITERATION_LIMIT, done)
        # next iterate: Halpern, or z~ where the LP restarts
        a = (k + 1.0) / (k + 2.0)
        XN, YN = a * (2.0 * XT - X) + XA / (k + 2.0), a * (2.0 * YT - Y) + YA / (k + 2.0)
        XAN, YAN, kn = XA, YA, k + 1.0
        if full or fresh:
            zero = k == 0
            due = (r <= 0.2 * r0) | ((rp >= 0) & (r <= 0.8 * r0) & (r > rp)) | (k > 0.36 * it)
            due = due & ~zero & full
            r0 = torch.where(zero, r, r0)
            if full:
                rp = torch.where(due, -1.0, r)
            else:
                rp = torch.where(zero, r, rp)
            if bool(due.any()):
                num, den = (YT - YA).norm(dim=0), (XT - XA).norm(dim=0)
                ok = (num > 1e-10) & (den > 1e-10)
                wn = torch.exp(0.5 * torch.log(torch.where(ok, num / den, w)) + 0.5 * torch.log(w))
                w = torch.where(due & ok, wn, w)
                XN, YN = torch.where(due, XT, XN), torch.where(due, YT, YN)
                XAN, YAN, kn = torch.where(due, XT, XA), torch.where(due, YT, YA), torch.where(due, 0.0, kn)
        if bool((done != 0).any()):
            q = torch.nonzero(done)[:, 0]
            ids = live[q].cpu().numpy()
            X_out[live[q]], Y_out[live[q]] = (XT[:, q] * t(dc)[:, None]).T, (YT[:, q] * t(dr)[:, None]).T
            status[ids], its[ids] = done[q].cpu().numpy(), it + 1
            kkt[ids] = torch.stack([gap[q], pri[q], dua[q], rel[q]], 1).cpu().numpy()
            obj[ids] = cx[q].cpu().numpy()
            s = torch.nonzero(done == 0)[:, 0]
            if not s.numel():
                break
            live, var, val, w, up, dn, ob, lo_j, hi_j, r0, rp, kn = (
                z[s] for z in (live, var, val, w, up, dn, ob, lo_j, hi_j, r0, rp, kn))
            XN, YN, XAN, YAN, cost = (z[:, s].contiguous() for z in (XN, YN, XAN, YAN, cost))
        X, Y, XA, YA, k = XN, YN, XAN, YAN, kn
    return {"X": X_out, "Y": Y_out, "status": status, "kkt": kkt, "obj": obj, "iters": its}


def exact(case, seed):
    o = _options(case)
    args = (case["C"], case["S"], case["tol"], o["dual_tol"], case["iters"], o["scaling"])
    if case["kind"] == "serve":
        # an LP's result does not depend on what runs beside it: one batch per base and kind
        bases, reqs = _inputs(case, seed)
        got = {}
        for bi, inst in enumerate(bases):
            for is_obj in (False, True):
                at = [i for i, (b, D) in enumerate(reqs) if b == bi and (D["kind"][0] == P.OBJ_UNIT) == is_obj]
                if not at:
                    continue
                D = np.concatenate([reqs[i][1] for i in at])
                # objective changes start from the base x with y = 0 and the default weight
                y0, w0 = (None, None) if is_obj else (inst["y"], np.full(len(D), _weight(inst)))
                r = _reference(inst, D, inst["x"], y0, w0, *args)
                cut = np.cumsum([len(reqs[i][1]) for i in at])[:-1]
                for q, i in enumerate(at):
                    got[i] = [np.split(r[key], cut)[q] for key in ("status", "iters", "obj")]
        return {key: np.concatenate([got[i][j] for i in range(len(reqs))])
                for j, key in enumerate(("statuses", "iters", "objs"))}
    inst, D = _inputs(case, seed)
    if case["kind"] == "branch":
        return _reference(inst, D, inst["x"], inst["y"], np.full(len(D), _weight(inst)), *args)
    return _reference(inst, D, None, None, None, *args)
