"""Blocks of iterations of small matrices in one launch (a workgroup per LP, or the
workgroups of an XCD per chunk of columns) against the step launches, bit for bit:
results, statuses, iteration counts, restart logs and last iterates.  Kernel timing
runs a solve on the step launches, which is the reference here."""
from __future__ import annotations

import ctypes as C

import numpy as np
import pytest

from gpu_common import cfg2_setup, make_ctx
from workloads import (choose_vars, make_cfg1, make_cfg2, make_facility, make_packing, make_setcover,
                       make_tiny, obbt_deltas)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2601_21990_amd.pdlpb as P
    return P


def _solve(ctx, D, tol, K, timing, warm=None):
    ctx.set_kernel_timing(timing)
    kw = {} if warm is None else dict(x_warm=warm.x, y_warm=warm.y, w_warm=np.full(len(D), warm.w))
    ctx.set_batch(D, **kw)
    ctx.solve(tol=tol, max_iters=K)
    out = ctx.get_batch()
    out["dobj"] = ctx.dual_objective()
    return out, [ctx.get_trace(j) for j in range(len(D))]


def _same(inst, D, tol, K, warm=None, **kw):
    with make_ctx(inst, **kw) as ctx:
        a, ta = _solve(ctx, D, tol, K, False, warm)
        b, tb = _solve(ctx, D, tol, K, True, warm)
        c, _ = _solve(ctx, D, tol, K, False, warm)     # the groups' words are clear again
    for key in a:
        assert np.array_equal(a[key], b[key], equal_nan=True), key
        assert np.array_equal(a[key], c[key], equal_nan=True), key
    for x, y in zip(ta, tb):
        assert np.array_equal(x["x_iter"], y["x_iter"]) and np.array_equal(x["y_iter"], y["y_iter"])
        assert x["w"] == y["w"] and x["restart_log"] == y["restart_log"]
    return a


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("make, B", [
    (lambda: make_tiny(3, m=3, n=5), 2),                # one wave a side, a few rows
    (make_cfg1, 6),                                     # empty rows and columns
    (lambda: make_cfg2(m=64, n=128), 5),                # whole waves
    (lambda: make_cfg2(m=65, n=143), 3),                # remainders of panels and waves
    (lambda: make_facility(F=6, C=24, k=4), 7),         # rows longer than the held indices
    (lambda: make_cfg2(m=200, n=500), 300),             # more LPs than compute units
], ids=["tiny", "empty", "64x128", "65x143", "long", "200x500"])
def test_solo(P, make, B, prec):
    inst = make()
    precision = P.MIXED32 if prec == "fp32" else P.FP64
    n = inst.n
    D = obbt_deltas(choose_vars(n, min(n, (B + 1) // 2), seed=B))[:B]
    _same(inst, D, 1e-5, 700, precision=precision)
    for K in (2, 65, 100):                              # limits at, after and inside a block
        _same(inst, D[:3], 0.0, K, precision=precision)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("m, n, B", [
    (2000, 5000, 1), (2000, 5000, 8),                   # one column per XCD
    (1037, 2611, 3),                                    # odd rows: slices and copies with remainders
    (2000, 5000, 9), (2000, 5000, 31), (2000, 5000, 64), (1500, 3701, 100), (1000, 2500, 128),
])
def test_grouped(P, m, n, B, prec):
    inst = make_cfg2(m=m, n=n)
    D = obbt_deltas(choose_vars(n, (B + 1) // 2, seed=B))[:B]
    precision = P.MIXED32 if prec == "fp32" else P.FP64
    _same(inst, D, 1e-4, 600, precision=precision, eval_every=32)
    _same(inst, D, 0.0, 45, precision=precision, eval_every=32, stop_every=8)


@pytest.mark.parametrize("stop", [0, 8])
def test_grouped_converged(P, stop):
    """Strong branching to the end: restarts, stops at every kind of test, an
    infeasible branch, compactions between the launches."""
    inst, lp, eta, base, D = cfg2_setup()
    _same(inst, D, 1e-4, 20000, warm=base, step_size=eta, eval_every=32, stop_every=stop)
    _same(inst, D[:5], 1e-6, 20000, warm=base, step_size=eta, eval_every=32, stop_every=stop)


@pytest.mark.parametrize("make", [lambda: make_facility(F=40, C=300), lambda: make_setcover(m=2000, n=4000),
                                  lambda: make_packing(m=400, n=900)], ids=["facility", "cover", "packing"])
@pytest.mark.parametrize("B", [6, 40])
def test_grouped_structured(P, make, B):
    """Columns of over a hundred entries, 0/1 matrices, diagonal scaling."""
    inst = make()
    D = obbt_deltas(choose_vars(inst.n, B // 2, seed=B))
    _same(inst, D, 1e-4, 500, scaling=1, dual_tol=1e-8)


@pytest.mark.parametrize("m, n, B, grouped", [
    (3200, 6500, 2, True), (3200, 6500, 12, True),      # row segments of one and two columns
    (5000, 9000, 3, True),
    (7000, 11000, 1, False), (7000, 11000, 4, False),   # the slices fit, but step launches are faster;
    (7000, 11000, 5, True), (7000, 11000, 12, True),    # not so with more columns
    (8000, 12000, 8, False),
])
def test_grouped_where_faster(P, m, n, B, grouped):
    """Grouped launches where they beat the step launches (only they take work vectors)."""
    inst = make_cfg2(m=m, n=n)
    D = obbt_deltas(choose_vars(n, (B + 1) // 2, seed=B))[:B]
    with make_ctx(inst, eval_every=32) as ctx:
        ctx.set_batch(D)
        before = ctx.device_bytes
        ctx.solve(tol=0.0, max_iters=33)
        assert (ctx.device_bytes > before) == grouped
    _same(inst, D, 1e-4, 100, eval_every=32)


class _NanAllocator:
    """Device memory of a caller's allocator, every word a NaN (FP64 and FP32); none
    while `full` is set."""

    def __init__(self, P):
        import torch
        self.live = {}
        self.full = False

        def alloc(nbytes, _user):
            if self.full:
                return None
            t = torch.full((int(nbytes),), 255, dtype=torch.uint8, device="cuda:0")
            torch.cuda.synchronize()
            self.live[t.data_ptr()] = t
            return t.data_ptr()

        def free(ptr, nbytes, _user):
            del self.live[int(ptr)]

        self.c_alloc, self.c_free = P.DEV_ALLOC(alloc), P.DEV_FREE(free)

    def install(self, opts):
        opts.dev_alloc = C.cast(self.c_alloc, C.c_void_p).value
        opts.dev_free = C.cast(self.c_free, C.c_void_p).value
        opts.alloc_user = None


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("m, n, B, sizes", [
    (2001, 5000, 64, (1, 15, 17, 31)),    # larger slices than the LDS holds; odd rows
    (1037, 2611, 9, (1, 12, 14, 18)),     # ... that still fit in larger groups
    (300, 701, 30, (1, 5, 11)),           # ... in most
    (2000, 5000, 1, (1, 13, 15)),         # one column: members of more rows than threads
    (1037, 2611, 3, (1, 5, 11, 15)),
])
def test_short_groups(P, m, n, B, sizes, prec):
    """Groups that close with fewer workgroups than planned (as beside other work on
    the device), on memory that holds NaN before its first use: the step launches'
    bits, whether the groups work or leave the iterations to step launches."""
    inst = make_cfg2(m=m, n=n)
    D = obbt_deltas(choose_vars(n, (B + 1) // 2, seed=B))[:B]
    precision = P.MIXED32 if prec == "fp32" else P.FP64
    fn = P.lib.pdlpb_group_launch
    fn.argtypes, fn.restype = [C.c_void_p, C.c_int32], C.c_int
    with make_ctx(inst, precision=precision, eval_every=32, stop_every=8) as ctx:
        ref, rt = _solve(ctx, D, 1e-4, 150, True)
    with make_ctx(inst, precision=precision, eval_every=32, stop_every=8, allocator=_NanAllocator(P)) as ctx:
        for size in sizes:
            assert fn(ctx._h, size) == P.OK
            print(f"short group m={m} n={n} B={B} {prec} size={size}", flush=True)
            got, gt = _solve(ctx, D, 1e-4, 150, False)
            for key in ref:
                assert np.array_equal(ref[key], got[key], equal_nan=True), (size, key)
            for x, y in zip(rt, gt):
                assert np.array_equal(x["x_iter"], y["x_iter"]) and np.array_equal(x["y_iter"], y["y_iter"])
                assert x["w"] == y["w"] and x["restart_log"] == y["restart_log"]


@pytest.mark.parametrize("B", [1, 40])
def test_no_memory_for_grouped(P, B):
    """A device with no memory left for the work vectors: the solve runs on step
    launches, and on grouped ones once there is memory again."""
    inst = make_cfg2(m=2000, n=5000)
    D = obbt_deltas(choose_vars(inst.n, (B + 1) // 2, seed=B))[:B]
    alloc = _NanAllocator(P)
    with make_ctx(inst, eval_every=32, allocator=alloc) as ctx:
        ref, _ = _solve(ctx, D, 1e-4, 200, True)
        before = ctx.device_bytes
        ctx.set_kernel_timing(False)
        for full in (True, False):
            alloc.full = full
            ctx.set_batch(D)
            ctx.solve(tol=1e-4, max_iters=200)
            alloc.full = False
            got = ctx.get_batch()
            assert (ctx.device_bytes > before) != full
            for key in got:
                assert np.array_equal(ref[key], got[key], equal_nan=True), (full, key)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("m, n, B", [
    (150, 400, 5),                                      # solo
    (1500, 3701, 3), (1500, 3701, 20),                  # staged; row segments
    (4001, 12001, 20),                                  # the row kernel
])
def test_not_finite(P, m, n, B, prec):
    """Iterates that overflow within a block of iterations (a step size far too large,
    some free variables among boxed ones): pads and empty slots of the persistent
    blocks and the row kernel add nothing to a sum that gathers infinities or NaN."""
    inst = make_cfg2(m=m, n=n)
    inst.l[::40], inst.u[::40] = -np.inf, np.inf
    D = obbt_deltas(choose_vars(n, (B + 1) // 2, seed=B))[:B]
    kw = dict(precision=P.MIXED32 if prec == "fp32" else P.FP64, eval_every=64,
              step_size=1e8 if prec == "fp64" else 1e3)
    budgets = (3, 4, 5, 6, 7, 8, 9, 10, 12, 16, 18, 19, 20, 21, 22, 24, 40)
    out = []
    for timing, shape in ((True, dict(tile_lanes=8, tile_vec=1)), (True, {}), (False, {})):
        with make_ctx(inst, **kw, **shape) as ctx:
            out.append([_solve(ctx, D, 1e-9, K, timing) for K in budgets])
    # some of the budgets end while part of the coordinates is finite
    bad = [np.mean(~np.isfinite(ref["X"])) for ref, _ in out[0]]
    assert bad[0] == 0.0 and bad[-1] > 0.0 and any(0.0 < b < 1.0 for b in bad), bad
    for run in out[1:]:
        for K, (ref, rt), (got, gt) in zip(budgets, out[0], run):
            for key in ref:
                assert np.array_equal(ref[key], got[key], equal_nan=True), (K, key)
            for x, y in zip(rt, gt):
                assert np.array_equal(x["x_iter"], y["x_iter"], equal_nan=True), K
                assert np.array_equal(x["y_iter"], y["y_iter"], equal_nan=True), K


def test_workgroup_cap(P):
    """A cap on the workgroups of a launch (max_blocks) holds for small matrices too:
    step launches, with the same bits."""
    inst = make_cfg2(m=2000, n=5000)
    D = obbt_deltas(choose_vars(inst.n, 20, seed=1))
    out = []
    for cap in (0, 16):
        with make_ctx(inst, eval_every=32, max_blocks=cap) as ctx:
            ctx.set_batch(D)
            before = ctx.device_bytes
            ctx.solve(tol=1e-4, max_iters=100)
            assert (ctx.device_bytes > before) == (cap == 0)
            out.append(ctx.get_batch())
    for key in out[0]:
        assert np.array_equal(out[0][key], out[1][key], equal_nan=True), key


def test_serving_releases_the_work_vectors(P):
    """A serving session holds none of a batch's grouped launches, whose scratch its own
    launches cannot use; a later batch gets them again."""
    inst = make_cfg2(m=2000, n=5000)
    D = obbt_deltas(choose_vars(inst.n, 20, seed=1))
    with make_ctx(inst, eval_every=32) as ctx, make_ctx(inst, eval_every=32) as fresh:
        a, _ = _solve(ctx, D, 1e-4, 100, False)
        for c in (ctx, fresh):
            c.serve_begin(64)
        assert ctx.device_bytes == fresh.device_bytes
        b, _ = _solve(ctx, D, 1e-4, 100, False)
    for key in a:
        assert np.array_equal(a[key], b[key], equal_nan=True), key


def test_beside_other_work(P):
    """Grouped solves while another thread's context holds compute units with solo
    blocks and step launches: groups may close short, results do not change."""
    import threading
    inst, other = make_cfg2(m=1500, n=3701), make_cfg2(m=200, n=500)
    D, E = obbt_deltas(choose_vars(3701, 20, seed=1)), obbt_deltas(choose_vars(500, 150, seed=2))
    stop, errors = threading.Event(), []
    with make_ctx(inst, eval_every=32) as ctx, make_ctx(other, eval_every=32) as busy:
        ref, _ = _solve(ctx, D, 1e-4, 400, True)
        want, _ = _solve(busy, E, 0.0, 900, True)

        def work():
            try:
                while not stop.is_set():
                    for timing in (False, True):
                        got, _ = _solve(busy, E, 0.0, 900, timing)
                        assert all(np.array_equal(want[k], got[k], equal_nan=True) for k in want)
            except Exception as e:      # noqa: BLE001 (reported by the main thread)
                errors.append(e)

        th = threading.Thread(target=work)
        th.start()
        try:
            for _ in range(10):
                got, _ = _solve(ctx, D, 1e-4, 400, False)
                for key in ref:
                    assert np.array_equal(ref[key], got[key], equal_nan=True), key
        finally:
            stop.set()
            th.join()
    assert not errors, errors


def test_two_contexts_at_once(P):
    """Two threads solve on grouped launches of one device: each gets its results."""
    import threading
    inst = [make_cfg2(rep=r, m=2000, n=5000) for r in range(2)]
    D = [obbt_deltas(choose_vars(5000, 12, seed=r)) for r in range(2)]
    ref, got = [], [None, None]
    ctx = [make_ctx(i, eval_every=32) for i in inst]
    for r in range(2):
        ref.append(_solve(ctx[r], D[r], 1e-4, 400, True)[0])

    def work(r):
        for _ in range(5):
            got[r] = _solve(ctx[r], D[r], 1e-4, 400, False)[0]

    th = [threading.Thread(target=work, args=(r,)) for r in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for r in range(2):
        for key in ref[r]:
            assert np.array_equal(ref[r][key], got[r][key], equal_nan=True), key
        ctx[r].close()
