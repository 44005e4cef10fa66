"""Batches whose blocks end inside, at and past a column tile (128 bytes per row):
every LP's results are, bit for bit, those it has in a batch of at most four LPs,
whose blocks are one narrow tile.  The row kernel of the steps against the kernels
that take any launch shape, bit for bit: every width it has, rows that fill, miss
and spill the entries a wave holds, 16 and 8 rows per wave."""
from __future__ import annotations

import numpy as np
import pytest

from gpu_common import make_ctx
from workloads import choose_vars, make_cfg1, make_cfg2, make_facility, make_packing, obbt_deltas

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_2601_21990_amd.pdlpb as P
    return P


def _solve(ctx, D, K):
    ctx.set_batch(D)
    ctx.solve(tol=1e-9, max_iters=K)
    out = ctx.get_batch()
    out["dobj"] = ctx.dual_objective()
    return out


def _pieces(inst, D, K, **kw):
    """The batch as a whole and in pieces of four, on the step launches."""
    with make_ctx(inst, **kw) as ctx:
        ctx.set_kernel_timing(True)
        whole = _solve(ctx, D, K)
        for i in range(0, len(D), 4):
            part = _solve(ctx, D[i:i + 4], K)
            for key in whole:
                assert np.array_equal(whole[key][i:i + 4], part[key], equal_nan=True), (key, i)


def _deltas(n, B):
    return obbt_deltas(choose_vars(n, min(n, (B + 1) // 2), seed=B))[:B]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("B", [15, 16, 17, 31, 32, 33, 48, 65, 151])
def test_widths(P, B, prec):
    inst = make_cfg2(m=300, n=700)
    _pieces(inst, _deltas(inst.n, B), 130, precision=P.MIXED32 if prec == "fp32" else P.FP64, eval_every=32)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("make, B", [
    (make_cfg1, 20),                                    # empty rows and columns
    (lambda: make_facility(F=6, C=24, k=4), 37),        # rows of very different lengths
], ids=["empty", "long"])
def test_shapes(P, make, B, prec):
    inst = make()
    D = _deltas(inst.n, B)
    _pieces(inst, D, 130, precision=P.MIXED32 if prec == "fp32" else P.FP64, eval_every=32)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("make, B", [
    (make_cfg1, 3),                                     # empty rows, a part of a wave
    (lambda: make_cfg2(m=97, n=211), 16),               # half a tile (FP32), a whole one (FP64)
    (lambda: make_cfg2(m=97, n=211), 31),               # odd widths: one slot per lane
    (lambda: make_cfg2(m=97, n=211), 34),               # two slots per lane in both
    (lambda: make_facility(F=4, C=600, k=4), 33),       # columns and rows of 600 entries among short ones
    (lambda: make_cfg2(m=3000, n=7000), 151),           # enough waves for 16 rows each
    (lambda: make_cfg2(m=16385, n=32770), 1),           # a lane per row, a remainder of a wave
    (lambda: make_cfg2(m=16385, n=32770), 2),           # a lane per row on one side
    (lambda: make_cfg2(m=30000, n=65537), 3),           # four columns, two lanes per row (FP64)
    (lambda: make_facility(F=4, C=4500, k=4), 1),       # a lane per row, rows of 4500 entries
], ids=["empty", "16", "31", "34", "spill", "many", "one", "two", "three", "one-spill"])
def test_row_kernel(P, make, B, prec):
    inst = make()
    D = _deltas(inst.n, B)
    kw = dict(precision=P.MIXED32 if prec == "fp32" else P.FP64, eval_every=32)
    out = []
    for shape in ({}, dict(tile_lanes=8, tile_vec=1)):
        with make_ctx(inst, **kw, **shape) as ctx:
            ctx.set_kernel_timing(True)
            out.append(_solve(ctx, D, 70))
    for key in out[0]:
        assert np.array_equal(out[0][key], out[1][key], equal_nan=True), key


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("B", [7, 9, 15, 17, 19, 29, 31, 33])
def test_row_kernel_odd_widths(P, B, prec):
    """Odd batches on the row kernel, the row stride padded to what a lane loads (blocks
    of that size, beside two result blocks a side): the bits of the kernels of any
    launch shape."""
    inst = make_cfg2(m=4001, n=12001)
    D = _deltas(inst.n, B)
    kw = dict(precision=P.MIXED32 if prec == "fp32" else P.FP64, eval_every=32)
    pad = 1 if B < 9 else 4 if prec == "fp32" and B > 16 else 2
    out, held = [], []
    for shape in ({}, dict(tile_lanes=8, tile_vec=1)):
        with make_ctx(inst, **kw, **shape) as ctx:
            ctx.set_kernel_timing(True)
            before = ctx.device_bytes
            out.append(_solve(ctx, D, 70))
            held.append(ctx.device_bytes - before)
    for key in out[0]:
        assert np.array_equal(out[0][key], out[1][key], equal_nan=True), key
    ld = -(-B // pad) * pad
    assert held[0] >= (4 * ld + 2 * B) * (inst.m + inst.n) * (4 if prec == "fp32" else 8)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("make, B", [
    (lambda: make_cfg2(m=20000, n=12001), 3),           # empty rows
    (lambda: make_cfg2(m=20000, n=12001), 16),
    (lambda: make_cfg2(m=20000, n=12001), 32),
    (lambda: make_facility(F=16, C=4000, k=4), 33),     # columns and rows of 1000 entries among short ones
    (make_facility, 20),                                # long rows side by side: 8 rows a wave,
    (make_facility, 33),                                # or the kernels of any launch shape (FP32)
    (make_facility, 130),
    (lambda: make_cfg2(m=4001, n=9999), 17),            # either side of the bound on small launches (FP32)
    (lambda: make_cfg2(m=4001, n=10001), 17),
    (lambda: make_cfg2(m=801, n=1999), 13),             # ... (FP64)
    (lambda: make_cfg2(m=801, n=2001), 13),
], ids=["empty3", "empty16", "empty32", "spill", "long20", "long33", "long130", "9999", "10001", "1999", "2001"])
def test_row_kernel_not_small(P, make, B, prec):
    """The row kernel where launches are not small, and at the line."""
    test_row_kernel(P, make, B, prec)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("m, n", [(63, 143), (64, 129), (1000, 2500), (33000, 66000)])
def test_row_evaluations(P, m, n, prec):
    """Evaluations with a lane per row (4 and 8 rows per chain, groups that end inside
    a panel) against the 64-slot kernel, which a batch of 40 takes."""
    inst = make_cfg2(m=m, n=n)
    D = _deltas(inst.n, 40)
    with make_ctx(inst, precision=P.MIXED32 if prec == "fp32" else P.FP64, eval_every=8) as ctx:
        ctx.set_kernel_timing(True)
        whole = _solve(ctx, D, 33)
        for i, j in ((0, 1), (1, 7), (7, 18)):
            part = _solve(ctx, D[i:j], 33)
            for key in whole:
                assert np.array_equal(whole[key][i:j], part[key], equal_nan=True), (key, i)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("m, n", [(33000, 66000), (66000, 33000), (65536, 65536)])
def test_evaluations_of_large_panels(P, m, n, prec):
    """Panels of 64 and 32 rows at widths that fill the row kernel's workgroups (four
    columns) and that leave it to the panel kernel, with stopping tests in between."""
    inst = make_cfg2(m=m, n=n)
    D = _deltas(inst.n, 40)
    with make_ctx(inst, precision=P.MIXED32 if prec == "fp32" else P.FP64, eval_every=8, stop_every=4) as ctx:
        ctx.set_kernel_timing(True)
        whole = _solve(ctx, D, 33)
        for i, j in ((0, 3), (3, 7), (7, 15), (15, 28)):
            part = _solve(ctx, D[i:j], 33)
            for key in whole:
                assert np.array_equal(whole[key][i:j], part[key], equal_nan=True), (key, i)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("m, n", [(63, 143), (600, 1399), (601, 1400), (1000, 2500), (1500, 3500), (1501, 3501)])
def test_evaluations_of_few_rows(P, m, n, prec):
    """Either side of the line between the panel kernel and the row kernel: one to 16
    columns, with stopping tests in between."""
    inst = make_cfg2(m=m, n=n)
    D = _deltas(inst.n, 40)
    with make_ctx(inst, precision=P.MIXED32 if prec == "fp32" else P.FP64, eval_every=8, stop_every=2) as ctx:
        ctx.set_kernel_timing(True)
        whole = _solve(ctx, D, 33)
        for i, j in ((0, 1), (1, 3), (3, 7), (7, 12), (12, 22), (22, 38)):
            part = _solve(ctx, D[i:j], 33)
            for key in whole:
                assert np.array_equal(whole[key][i:j], part[key], equal_nan=True), (key, i)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("F, C", [(20, 200), (100, 1000), (200, 2000)])
def test_evaluations_of_long_rows(P, F, C, prec):
    """Long rows side by side: the widths that each of the evaluation kernels takes."""
    inst = make_facility(F=F, C=C, k=8)
    D = _deltas(inst.n, 40)
    with make_ctx(inst, precision=P.MIXED32 if prec == "fp32" else P.FP64, eval_every=8, stop_every=4) as ctx:
        ctx.set_kernel_timing(True)
        whole = _solve(ctx, D, 33)
        for i, j in ((0, 1), (1, 3), (3, 7), (7, 15), (15, 31)):
            part = _solve(ctx, D[i:j], 33)
            for key in whole:
                assert np.array_equal(whole[key][i:j], part[key], equal_nan=True), (key, i)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("B", [16, 17, 20, 21, 32, 33, 36, 40, 41, 49, 64, 65])
def test_dense_rows(P, B, prec):
    """Columns of 40 and rows of 100 entries, past what the row kernel takes: batches whose
    last storage tile
    is up to a quarter full and just past that, against narrow row groups, bit for bit."""
    inst = make_packing(m=200, n=500, k=40)
    D = _deltas(inst.n, B)
    kw = dict(precision=P.MIXED32 if prec == "fp32" else P.FP64, eval_every=32)
    out = []
    for shape in ({}, dict(tile_lanes=8, tile_vec=1)):
        with make_ctx(inst, **kw, **shape) as ctx:
            ctx.set_kernel_timing(True)
            out.append(_solve(ctx, D, 70))
    for key in out[0]:
        assert np.array_equal(out[0][key], out[1][key], equal_nan=True), key
